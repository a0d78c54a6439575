// The persistent streaming GEMV (gemv_stream_kernel.h) on codes of 6 bits, both formats.
#include "gemv_stream_kernel.h"

namespace uniql {

hipError_t launch_w6_gemv_stream(const LinearArgs& a, hipStream_t stream, bool* done) { return gemv::stream_wide<6>(a, stream, done); }

}  // namespace uniql
