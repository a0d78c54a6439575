// The ring kernel (ring_kernel.h) on 3-bit codes, fp16.
#include "ring_dispatch.h"

namespace uniql {
hipError_t launch_ring_w3(const LinearArgs* p, hipStream_t stream) { return ring_linears<3, false>(p, 1, stream); }
}  // namespace uniql
