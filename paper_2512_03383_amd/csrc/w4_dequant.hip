// Bit-exact dequantisation of the kept sub-matrix: w = RN_fp16((q - z) * s), or RN_bf16 when scales and
// output are bfloat16.
// The product of the small integer (q - z) and the 11-bit (8-bit) significand of s is
// exact in fp32, so the single fp32 -> 16-bit conversion is the only rounding.
// (Written with scalar fp32 arithmetic on purpose: it is the independent check
// of the packed-fp16 dequantisation used inside the GEMV / GEMM kernels.)
#include "common.h"

namespace uniql {

// Bound by the output: 2 bytes written per half byte read.  A lane takes a word of a chunk, so a store instruction writes up to 1 KB
// of consecutive output and a load reads 256 bytes of codes, U chunks in flight per wave: 1 << CL of each of U >> CL rows.  Rows
// of at most 32 words (NARROW) share chunks: 1 << lanes_log2 lanes each.
// 10752 x 4096 kept: 24.4 us with eight chunks in flight (four 24.9, two 28.9; a thread per word of the whole matrix with eight 2-byte
// stores 62).  A wave to a row whatever its length left lanes idle on narrow rows and the chip on few long ones:
// 343750 x 128 102 us, so 24.4, 13 x 18944 11.9, so 3.5 (from graphs over six copies of the matrix; 10752 x 4096 in that way 20).
// A word's eight columns are written at once when all are kept; the word that holds the last kept columns of the row or of a
// segment, and column rules whose segments are not whole words, go element by element.
template <bool BF16, int U, int CL, bool NARROW>
__global__ __launch_bounds__(256) void w4_dequant_kernel(LinearArgs a, int lanes_log2, int row_step, int part_step) {
  constexpr int CH = 1 << CL;             // chunks of a row per turn
  constexpr bool one_row = CH == U && !NARROW;
  static_assert(CH <= U && (!NARROW || CL == 0), "whole rows per turn");
  const KeepMap& km = a.km;
  // a scalar wave number makes the addresses of several rows scalar (114583 x 384: 24.8 us, 27.8 from vectors); one row has a
  // single base, and with that formed once per turn a vector is no slower (10752 x 4096, 25 % rate: 61.9 us with the whole step, so 61.7)
  const int lane = threadIdx.x & 63, wave = one_row ? (int)(threadIdx.x >> 6) : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int words_span = (km.k_span + 7) >> 3;
  const int words_per_row = a.K_total >> 3;
  const int groups_per_row = a.K_total / kGroup;
  const int wph = a.il_heads > 0 ? words_per_row / a.il_heads : 1;
  const bool whole_words = km.cs_stride % 8 == 0;   // (a prefix: stride 0)
  const int ll = NARROW ? lanes_log2 : 6, lane_row = lane >> ll, lane_word = lane & ((1 << ll) - 1);
  const int turn_rows = (U >> CL) << (6 - ll);
  // the walk over rows, and over the turns of a long row (by steps that come with the other arguments: the grid's size would be a
  // load of its own on the way to the first word)
  for (long long r0 = ((long long)blockIdx.x * 4 + wave) * turn_rows; r0 < km.n_keep; r0 += row_step)
    for (int part0 = (int)blockIdx.y * CH; part0 * 64 < words_span; part0 += part_step) {
      uint32_t word[U], sb[U], zb[U];
      const size_t row1 = one_row ? (size_t)stored_row(km, (int)r0) : 0;   // of the whole turn
#pragma unroll
      for (int u = 0; u < U; ++u) {
        // (a row or word past the last one reads the last one)
        const long long rc = r0 + ((u >> CL) << (6 - ll)) + (NARROW ? lane_row : 0);
        const int w = min((part0 + u % CH) * 64 + lane_word, words_span - 1);
        const size_t row = one_row ? row1 : (size_t)stored_row(km, rc < km.n_keep ? (int)rc : km.n_keep - 1);
        // w counts words in column order; a head-interleaved row stores word (h, d / 8) at (d / 8) * H + h
        int ws = w;
        if (a.il_heads > 0) {
          const int h = w / wph;
          ws = (w - h * wph) * a.il_heads + h;
        }
        word[u] = (a.qweight + row * words_per_row)[ws];
        sb[u] = (a.scales + row * groups_per_row)[w >> 4];
        zb[u] = a.zeros ? (a.zeros + row * groups_per_row)[w >> 4] : 8;   // no zero points: the symmetric scheme
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const long long rc = r0 + ((u >> CL) << (6 - ll)) + (NARROW ? lane_row : 0);
        const int w = (part0 + u % CH) * 64 + lane_word;
        if (one_row) {
          if (w >= words_span) break;
        } else if (rc >= km.n_keep || w >= words_span) {
          continue;
        }
        const float s = in16<BF16>(__builtin_bit_cast(half_t, (uint16_t)sb[u]));
        const int z = (int)zb[u];
        uint16_t o[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] = __builtin_bit_cast(uint16_t, out16<BF16>((float)((int)((word[u] >> (4 * j)) & 15u) - z) * s));
        half_t* out = a.y + (size_t)rc * km.k_keep;
        int kc = 8 * w, nk = km.k_keep - kc, off = kc;   // compact column of the first one, kept columns from there, place in the segment
        if (km.cs_stride != 0) {
          const int seg = kc / km.cs_stride;
          off = kc - seg * km.cs_stride;
          nk = km.cs_keep - off;
          kc = seg * km.cs_keep + min(off, km.cs_keep);
        }
        if (whole_words && nk >= 8) {
          typedef uint32_t u32x4_u2 __attribute__((ext_vector_type(4), aligned(2)));
          u32x4_u2 v;
#pragma unroll
          for (int j = 0; j < 4; ++j) v[j] = o[2 * j] | ((uint32_t)o[2 * j + 1] << 16);
          *reinterpret_cast<u32x4_u2*>(out + kc) = v;
        } else if (whole_words) {
#pragma unroll
          for (int j = 0; j < 8; ++j)
            if (j < nk) out[kc + j] = __builtin_bit_cast(half_t, o[j]);
        } else {
          // (a word may hold the end of one segment and the beginning of the next)
          half_t* to = out + kc;
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            if (off < km.cs_keep) *to++ = __builtin_bit_cast(half_t, o[j]);
            off = off + 1 == km.cs_stride ? 0 : off + 1;
          }
        }
      }
    }
}

template <bool BF16, int U, int CL, bool NARROW>
static hipError_t launch_dequant_cfg(const LinearArgs& a, int lanes_log2, hipStream_t stream) {
  const int chunks = (a.km.k_span + 511) / 512, turn_rows = (U >> CL) << (6 - (NARROW ? lanes_log2 : 6));
  long long x = (((long long)a.km.n_keep + turn_rows - 1) / turn_rows + 3) / 4, y = (chunks + (1 << CL) - 1) >> CL;
  if (x > 65536) x = 65536;
  if (y > 65535) y = 65535;
  hipLaunchKernelGGL((w4_dequant_kernel<BF16, U, CL, NARROW>), dim3((unsigned)x, (unsigned)y), dim3(256), 0, stream, a, lanes_log2,
                     (int)x * 4 * turn_rows, (int)y << CL);
  return hipGetLastError();
}

template <bool BF16, int U>
static hipError_t launch_dequant(const LinearArgs& a, hipStream_t stream) {
  const int words = (a.km.k_span + 7) >> 3;
  int lanes_log2 = 0;
  while (lanes_log2 < 6 && (1 << lanes_log2) < words) ++lanes_log2;
  if (lanes_log2 < 6) return launch_dequant_cfg<BF16, U, 0, true>(a, lanes_log2, stream);
  if constexpr (U >= 8) {
    if (words > 256) return launch_dequant_cfg<BF16, U, 3, false>(a, 6, stream);
    if (words > 128) return launch_dequant_cfg<BF16, U, 2, false>(a, 6, stream);
  }
  if constexpr (U >= 2) {
    if (words > 64) return launch_dequant_cfg<BF16, U, 1, false>(a, 6, stream);
  }
  return launch_dequant_cfg<BF16, U, 0, false>(a, 6, stream);
}

template <bool BF16>
static hipError_t launch_dequant_fmt(const LinearArgs& a, hipStream_t stream) {
  const long long chunks = ((long long)a.km.n_keep * ((a.km.k_span + 7) >> 3) + 63) >> 6;
  // chunks in flight: eight where that leaves every SIMD two waves and more, fewer on more waves otherwise (44 / 4.2 / 0.26 million
  // codes of 4096 columns: eight 20.2 / 6.1 / 5.0 us, two 22.4 / 5.7 / 4.2, one 28.9 / 6.4 / 4.1)
  if (chunks >= 16384) return launch_dequant<BF16, 8>(a, stream);
  return chunks >= 4096 ? launch_dequant<BF16, 2>(a, stream) : launch_dequant<BF16, 1>(a, stream);
}

hipError_t launch_w4_dequant(const LinearArgs& a, hipStream_t stream) {
  return a.bf16 ? launch_dequant_fmt<true>(a, stream) : launch_dequant_fmt<false>(a, stream);
}

// Rows of a quantised table gathered by token id: out[i][:] = dequantised row ids[i].
// A wave handles one (token, 2048-column chunk): a lane reads 16 bytes of codes and the scale and
// zero point of its group, dequantises with the packed path of the GEMV, puts the 32 halves back
// into column order and writes 64 contiguous bytes.  Rows are K_total wide (the hidden dimension
// is never pruned).  BF16: the table's scales and the output are bfloat16 (fp32 arithmetic, subtract then
// multiply, so that a zero weight has the sign of (q - z) * s as in the fp16 path).
template <bool BF16>
__global__ __launch_bounds__(256) void w4_embedding_kernel(const uint32_t* qweight, const uint16_t* scales,
                                                           const uint8_t* zeros, int K_total, const int32_t* ids,
                                                           int n, half_t* out, long long ld) {
  const int lane = threadIdx.x & 63;
  const int chunks = (K_total + 2047) / 2048;
  const long long item = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);   // (token, chunk)
  if (item >= (long long)n * chunks) return;
  const int tok = (int)(item / chunks), c = (int)(item - (long long)tok * chunks);
  const int k0 = c * 2048 + lane * 32;
  if (k0 >= K_total) return;                      // K_total is a multiple of 128: a lane's 32 columns are all in or all out
  const size_t row = (size_t)ids[tok];
  const uint4 w = *reinterpret_cast<const uint4*>(qweight + row * (size_t)(K_total >> 3) + (k0 >> 3));
  const size_t g = row * (size_t)(K_total / kGroup) + (k0 >> 7);
  const uint32_t z = zeros ? zeros[g] : 8u;
  const typename GroupOf<BF16>::type gq = make_group<BF16>(scales[g], z);
  const Magic mg = make_magic();
  const uint32_t words[4] = {w.x, w.y, w.z, w.w};
  uint4* dst = reinterpret_cast<uint4*>(out + (size_t)tok * ld + k0);   // 16-byte aligned: checked by the host
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    uint4 d;                                      // (w0,w4) (w1,w5) (w2,w6) (w3,w7)
    if constexpr (BF16) d = dequant_word_bf16<true>(words[q], gq, (float)z);
    else d = dequant_word4<false>(words[q], gq, mg);
    const uint32_t a = d.x, b = d.y, cc = d.z, e = d.w;
    dst[q] = make_uint4(__builtin_amdgcn_perm(b, a, 0x05040100u), __builtin_amdgcn_perm(e, cc, 0x05040100u),
                        __builtin_amdgcn_perm(b, a, 0x07060302u), __builtin_amdgcn_perm(e, cc, 0x07060302u));
  }
}

hipError_t launch_w4_embedding(const uint32_t* qweight, const uint16_t* scales, const uint8_t* zeros, int K_total,
                               const int32_t* ids, int n, half_t* out, long long ld, int bf16, hipStream_t stream) {
  const long long items = (long long)n * ((K_total + 2047) / 2048);
  const long long blocks = (items + 3) / 4;
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  if (bf16)
    hipLaunchKernelGGL(w4_embedding_kernel<true>, dim3((unsigned)blocks), dim3(256), 0, stream, qweight, scales, zeros,
                       K_total, ids, n, out, ld);
  else
    hipLaunchKernelGGL(w4_embedding_kernel<false>, dim3((unsigned)blocks), dim3(256), 0, stream, qweight, scales, zeros,
                       K_total, ids, n, out, ld);
  return hipGetLastError();
}

// Compact copy of the kept channels.  Output row r' is stored row stored_row(r'); output group g' is source
// group (g' / gps_out) * gps_src + g' % gps_out (gps_out = 0: groups stay in place).  A thread moves one
// 16-byte unit (32 codes, a quarter of a group); the thread of a group's first unit also moves the
// group's scale and zero point.  Rows are contiguous on both sides, so the copy streams.
__global__ __launch_bounds__(256) void w4_repack_kernel(RepackArgs a) {
  const int units_out = a.K_out >> 5;
  const long long total = (long long)a.km.n_keep * units_out;
  const int units_src = a.K_total >> 5;
  const int groups_src = a.K_total / kGroup, groups_out = a.K_out / kGroup;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    const int rc = (int)(i / units_out);
    const int u = (int)(i - (long long)rc * units_out);
    const int go = u >> 2;
    const int g = a.gps_out ? (go / a.gps_out) * a.gps_src + go % a.gps_out : go;
    const size_t row = (size_t)stored_row(a.km, rc);
    const uint4* src = reinterpret_cast<const uint4*>(a.qweight) + row * units_src + (size_t)g * 4 + (u & 3);
    reinterpret_cast<uint4*>(a.out_qweight)[(size_t)rc * units_out + u] = *src;
    if ((u & 3) == 0) {
      a.out_scales[(size_t)rc * groups_out + go] = a.scales[row * groups_src + g];
      if (a.zeros) a.out_zeros[(size_t)rc * groups_out + go] = a.zeros[row * groups_src + g];
    }
  }
}

// Words of every row from head-major [heads][words per head] to [words per head][heads], or back (INV).  A thread
// moves one word; consecutive threads write consecutive words (the reads stride: the pass runs once per matrix).
template <bool INV>
__global__ __launch_bounds__(256) void w4_interleave_kernel(const uint32_t* __restrict__ qweight, uint32_t* __restrict__ out,
                                                            long long total, int words_per_row, int heads) {
  const int wph = words_per_row / heads;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (long long)gridDim.x * blockDim.x) {
    const long long row = i / words_per_row;
    const int wo = (int)(i - row * words_per_row);    // output word
    int src;
    if constexpr (INV) {                              // wo = h * wph + d / 8
      const int h = wo / wph, db = wo - h * wph;
      src = db * heads + h;
    } else {                                          // wo = (d / 8) * heads + h
      const int db = wo / heads, h = wo - db * heads;
      src = h * wph + db;
    }
    out[i] = qweight[row * words_per_row + src];
  }
}

hipError_t launch_w4_interleave(const uint32_t* qweight, uint32_t* out, int N_total, int K_total, int heads, bool inverse,
                                hipStream_t stream) {
  const long long total = (long long)N_total * (K_total >> 3);
  long long blocks = (total + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) blocks = 1;
  if (inverse)
    hipLaunchKernelGGL(w4_interleave_kernel<true>, dim3((unsigned)blocks), dim3(256), 0, stream, qweight, out, total, K_total >> 3, heads);
  else
    hipLaunchKernelGGL(w4_interleave_kernel<false>, dim3((unsigned)blocks), dim3(256), 0, stream, qweight, out, total, K_total >> 3, heads);
  return hipGetLastError();
}

hipError_t launch_w4_repack(const RepackArgs& a, hipStream_t stream) {
  const long long total = (long long)a.km.n_keep * (a.K_out >> 5);
  long long blocks = (total + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(w4_repack_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, a);
  return hipGetLastError();
}

}  // namespace uniql
