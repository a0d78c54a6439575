// The 8-bit bfloat16 instantiations of pipe_kernel.h.
#include "pipe_dispatch.h"

namespace uniql {

hipError_t launch_pipe_w8_bf16(const LinearArgs* p, int n, hipStream_t stream) { return pipe_linears<8, true>(p, n, stream); }

}  // namespace uniql
