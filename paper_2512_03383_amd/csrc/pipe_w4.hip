// The 4-bit fp16 instantiations of pipe_kernel.h.
#include "pipe_dispatch.h"

namespace uniql {

hipError_t launch_pipe_w4(const LinearArgs* p, int n, hipStream_t stream) { return pipe_linears<4, false>(p, n, stream); }

}  // namespace uniql
