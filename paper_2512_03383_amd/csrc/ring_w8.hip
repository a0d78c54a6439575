// The ring kernel (ring_kernel.h) on 8-bit codes, fp16.
#include "ring_dispatch.h"

namespace uniql {
hipError_t launch_ring_w8(const LinearArgs* p, hipStream_t stream) { return ring_linears<8, false>(p, 1, stream); }
}  // namespace uniql
