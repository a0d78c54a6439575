// The ring kernel (ring_kernel.h) on 6-bit codes, bfloat16.
#include "ring_dispatch.h"

namespace uniql {
hipError_t launch_ring_w6_bf16(const LinearArgs* p, hipStream_t stream) { return ring_linears<6, true>(p, 1, stream); }
}  // namespace uniql
