// The 6-bit fp16 instantiations of pipe_kernel.h.
#include "pipe_dispatch.h"

namespace uniql {

hipError_t launch_pipe_w6(const LinearArgs* p, int n, hipStream_t stream) { return pipe_linears<6, false>(p, n, stream); }

}  // namespace uniql
