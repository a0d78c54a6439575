// The ring kernel (ring_kernel.h) on 4-bit codes, fp16.
#include "ring_dispatch.h"

namespace uniql {
hipError_t launch_ring_w4(const LinearArgs* p, int n, hipStream_t stream) { return ring_linears<4, false>(p, n, stream); }
hipError_t launch_ring_glu(const LinearArgs* p, hipStream_t stream) { return ring_glu<false>(p, stream); }
}  // namespace uniql
