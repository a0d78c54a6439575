// The persistent streaming GEMV (gemv_stream_kernel.h) on codes of 8 bits, both formats; what the widths have in common on the host.
#include "gemv_stream_kernel.h"

namespace uniql {

hipError_t launch_w8_gemv_stream(const LinearArgs& a, hipStream_t stream, bool* done) { return gemv::stream_wide<8>(a, stream, done); }

int wide_walk_rows(const LinearArgs& a) {
  return gemv::stream_wide_takes(a) ? gemv::stream_rows(gemv::row_tiles(a.km.k_span), false) : 0;
}

}  // namespace uniql
