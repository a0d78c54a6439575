// The 4-bit bfloat16 instantiations of pipe_kernel.h.
#include "pipe_dispatch.h"

namespace uniql {

hipError_t launch_pipe_w4_bf16(const LinearArgs* p, int n, hipStream_t stream) { return pipe_linears<4, true>(p, n, stream); }

}  // namespace uniql
