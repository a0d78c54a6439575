// The ring kernel (ring_kernel.h) on 4-bit codes, bfloat16.
#include "ring_dispatch.h"

namespace uniql {
hipError_t launch_ring_w4_bf16(const LinearArgs* p, int n, hipStream_t stream) { return ring_linears<4, true>(p, n, stream); }
hipError_t launch_ring_glu_bf16(const LinearArgs* p, hipStream_t stream) { return ring_glu<true>(p, stream); }
}  // namespace uniql
