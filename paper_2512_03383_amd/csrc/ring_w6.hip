// The ring kernel (ring_kernel.h) on 6-bit codes, fp16.
#include "ring_dispatch.h"

namespace uniql {
hipError_t launch_ring_w6(const LinearArgs* p, hipStream_t stream) { return ring_linears<6, false>(p, 1, stream); }
}  // namespace uniql
