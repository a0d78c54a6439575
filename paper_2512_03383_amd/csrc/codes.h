// Codes of 8, 6, 4 and 3 bits as MFMA weight operands whose columns are in memory order (pipe_kernel.h).
//
// A lane holds the 32 columns of one k-slot of one group of one row: BITS 32-bit words, whole for every width (32 codes
// of BITS bits).  Step t (0..3) of the group multiplies the eight columns 8 t .. 8 t + 7 of the slot, and the operand holds
// them in order, so that the activations need no permutation on their way into LDS.
//
// As in the unpack of common.h a masked word OR-ed with an fp16 exponent pattern is a pair of exact fp16 numbers base + q
// (the subtraction of base + z is exact too); the two members of a pair may sit at different bit positions of their 16-bit
// halves and then take different exponents (1024, 128, 64 or 8: a code at bit 0, 3, 4 or 7).  Vector instructions per
// eight codes (fp16; bfloat16 below):
//   4 bits  16: a byte permute puts codes 0..3 (4..7) into both halves, code 2 j at bit 0 of the low one, 2 j + 1 at bit 4 of the high
//   3 bits  16: likewise, bytes 0 1 | 0 1 and 1 2 | 1 2 of the eight codes' three bytes, code positions 0 | 3 and 4 | 7
//   6 bits  20: pairs (j, j + 4) as two byte permutes of the six bytes, then four permutes put the weights in order
//   8 bits  12: a byte permute with a register of 0x64 bytes makes (1024 + q, 1024 + q') of neighbouring codes
//
// fp16 weight: (pair - (base + z)) * s in packed fp16, one rounding.  bfloat16: fma(member, s, -(base + z) s) in fp32 with
// the fp16 operand read in place (exact: the products and their difference fit 24 bits), then a packed conversion, one
// rounding; the members are converted one by one, so any order costs the same and the cheaper pairs (j, j + 4) of common.h
// serve 4 and 6 bits.  The constant (base + z) s overflows from scales of 2^128 / 1279 on where a weight need not, so a group
// with such a scale takes the wide form (member - (base + z)) * s, exact up to the rounding as well and two instructions a
// code; kScaleWide tells.
#pragma once
#include "common.h"

namespace uniql {

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

// words that hold T steps (T * BITS bytes) of a slot, the first one at byte 0
template <int BITS, int T>
struct RawCodes {
  uint32_t w[(T * BITS + 3) / 4];
};

// The codes of steps q T .. q T + T - 1 of a slot in LDS (q the same for the whole wave; 4-byte aligned address): eight codes
// are BITS bytes, so the window may start inside a word and is then shifted down.
template <int BITS, int T>
__device__ __forceinline__ RawCodes<BITS, T> read_codes(const unsigned char* slot, int q) {
  RawCodes<BITS, T> o;
  constexpr int N = (T * BITS + 3) / 4;
  if constexpr (T * BITS % 4 == 0) {
    const unsigned char* p = slot + q * (T * BITS);
    if constexpr (N == 4 && BITS == 4) {
      const uint4 v = *reinterpret_cast<const uint4*>(p);
      o.w[0] = v.x; o.w[1] = v.y; o.w[2] = v.z; o.w[3] = v.w;
    } else if constexpr (N % 2 == 0) {
#pragma unroll
      for (int i = 0; i < N; i += 2) {
        const u32x2_t v = *reinterpret_cast<const u32x2_t*>(p + 4 * i);
        o.w[i] = v.x; o.w[i + 1] = v.y;
      }
    } else {
#pragma unroll
      for (int i = 0; i < N; ++i) o.w[i] = *reinterpret_cast<const uint32_t*>(p + 4 * i);
    }
  } else {
    const int b = q * (T * BITS), sh = (b & 3) * 8;
    const uint32_t* p = reinterpret_cast<const uint32_t*>(slot + (b & ~3));
    uint32_t v[N + 1];
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = p[i];
    // (the word behind the window: only for a window that ends in it, which is never the slot's last)
    v[N] = (b & 3) * 8 + T * BITS * 8 > 32 * N ? p[N] : 0u;
#pragma unroll
    for (int i = 0; i < N; ++i) o.w[i] = __builtin_amdgcn_alignbit(v[i + 1], v[i], sh);
  }
  return o;
}

// exponent patterns and bases of the pair classes; class and columns of pair j of a step
template <int BITS, bool BF16>
struct CodeForm {
  static constexpr bool kFar = BITS == 6 || (BITS == 4 && BF16);   // pairs (j, j + 4); else (2 j, 2 j + 1)
  // 4 bits: (1024 | 64) or, far, 1024 and 64 alternating; 3 bits: (1024 | 128) for codes 0..3, (64 | 8) for 4..7; 6 bits: 1024
  // for pair 0, else 64; 8 bits: 1024
  static constexpr uint32_t kA = BITS == 8 || kFar ? 0x64006400u : (BITS == 4 ? 0x54006400u : 0x58006400u);
  static constexpr uint32_t kB = BITS == 3 ? 0x48005400u : 0x54005400u;
  static constexpr int kAlo = 0, kAhi = BITS == 8 || kFar ? 0 : (BITS == 4 ? 4 : 3);   // bit of the code in its half
  static constexpr int kBlo = 4, kBhi = BITS == 3 ? 7 : 4;
  static constexpr bool kOneClass = BITS == 8 || (BITS == 4 && !kFar);
  static constexpr bool is_b(int j) { return kOneClass ? false : (BITS == 6 ? j > 0 : (BITS == 3 ? j > 1 : (j & 1) != 0)); }
};

struct CodeMagic {
  uint32_t a, b;   // exponent patterns in VGPRs (8 bits: a = four bytes 0x64)
};
template <int BITS, bool BF16>
__device__ __forceinline__ CodeMagic make_code_magic() {
  CodeMagic m = {BITS == 8 ? 0x64646464u : CodeForm<BITS, BF16>::kA, CodeForm<BITS, BF16>::kB};
  asm volatile("" : "+v"(m.a), "+v"(m.b));
  return m;
}

// constants of one (row, group)
template <int BITS, bool BF16> struct CodeGroup;
template <int BITS> struct CodeGroup<BITS, false> {
  half2_t za, zb, s2;   // base + z of the two classes, scale
};
template <int BITS> struct CodeGroup<BITS, true> {
  float s, nalo, nahi, nblo, nbhi;   // scale, -(base + z) s of the two classes and halves (wide: base + z)
};

// bits of the smallest bfloat16 scale in magnitude, 2^117, from which on (1024 + z) s may overflow (1279 * 2^117 < 2^128);
// infinities and NaN lie above it
constexpr uint32_t kScaleWide = (127u + 117u) << 7;

template <int BITS, bool BF16, bool WIDE = false>
__device__ __forceinline__ CodeGroup<BITS, BF16> make_code_group(uint32_t sbits, uint32_t z) {
  typedef CodeForm<BITS, BF16> F;
  CodeGroup<BITS, BF16> g;
  if constexpr (BF16) {
    // a code at bit p of its half comes with the base 1024 / 2^p
    g.s = __builtin_bit_cast(float, sbits << 16);
    const float zf = (float)z, f = WIDE ? 1.f : -g.s;
    g.nalo = (1024.f / (1 << F::kAlo) + zf) * f;
    g.nahi = (1024.f / (1 << F::kAhi) + zf) * f;
    g.nblo = (1024.f / (1 << F::kBlo) + zf) * f;
    g.nbhi = (1024.f / (1 << F::kBhi) + zf) * f;
  } else {
    g.za = as_half2((z << F::kAlo) | (z << (16 + F::kAhi)) | F::kA);
    g.zb = F::kOneClass ? g.za : as_half2((z << F::kBlo) | (z << (16 + F::kBhi)) | F::kB);
    g.s2 = as_half2(sbits | (sbits << 16));
  }
  return g;
}

// a group's constants where `kept` is all ones, those of a scale of zero where it is zero
template <int BITS>
__device__ __forceinline__ CodeGroup<BITS, false> mask_code_group(const CodeGroup<BITS, false>& g, uint32_t kept) {
  return {g.za, g.zb, as_half2(as_u32(g.s2) & kept)};
}
template <int BITS>
__device__ __forceinline__ CodeGroup<BITS, true> mask_code_group(const CodeGroup<BITS, true>& g, uint32_t kept) {
  auto m = [&](float f) { return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, f) & kept); };
  return {m(g.s), m(g.nalo), m(g.nahi), m(g.nblo), m(g.nbhi)};
}

// the four pairs base + q of step t of the window
template <int BITS, bool BF16, int T>
__device__ __forceinline__ void code_pairs(const RawCodes<BITS, T>& r, int t, const CodeMagic& m, uint32_t (&p)[4]) {
  if constexpr (BITS == 4 && BF16) {
    const uint32_t w = r.w[t], w8 = w >> 8;
    p[0] = and_or(w, 0x000F000Fu, m.a);
    p[1] = and_or(w, 0x00F000F0u, m.b);
    p[2] = and_or(w8, 0x000F000Fu, m.a);
    p[3] = and_or(w8, 0x00F000F0u, m.b);
  } else if constexpr (BITS == 4) {
    const uint32_t w = r.w[t];
    const uint32_t v = __builtin_amdgcn_perm(w, w, 0x01000100u), u = __builtin_amdgcn_perm(w, w, 0x03020302u);
    p[0] = and_or(v, 0x00F0000Fu, m.a);
    p[1] = and_or(v >> 8, 0x00F0000Fu, m.a);
    p[2] = and_or(u, 0x00F0000Fu, m.a);
    p[3] = and_or(u >> 8, 0x00F0000Fu, m.a);
  } else if constexpr (BITS == 8) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const uint32_t w = r.w[2 * t + i];
      p[2 * i] = __builtin_amdgcn_perm(m.a, w, 0x04010400u);
      p[2 * i + 1] = __builtin_amdgcn_perm(m.a, w, 0x04030402u);
    }
  } else if constexpr (BITS == 6) {
    const int i = (6 * t) >> 2;
    const uint32_t o = (6 * t) & 3;          // byte of the first code in word i: 0 or 2
    const uint32_t lo = r.w[i], hi = r.w[i + 1 < (6 * T + 3) / 4 ? i + 1 : i];
    const uint32_t v = __builtin_amdgcn_perm(hi, lo, (o) | ((o + 1) << 8) | ((o + 3) << 16) | ((o + 4) << 24));
    const uint32_t u = __builtin_amdgcn_perm(hi, lo, (o + 1) | ((o + 2) << 8) | ((o + 4) << 16) | ((o + 5) << 24));
    p[0] = and_or(v, 0x003F003Fu, m.a);
    p[1] = and_or(v >> 2, 0x03F003F0u, m.b);
    p[2] = and_or(u, 0x03F003F0u, m.b);
    p[3] = and_or(u >> 6, 0x03F003F0u, m.b);
  } else {
    static_assert(BITS == 3, "codes of 8, 6, 4 or 3 bits");
    const int i = (3 * t) >> 2;
    const uint32_t o = (3 * t) & 3, lo = r.w[i], hi = r.w[i + 1 < (3 * T + 3) / 4 ? i + 1 : i];
    const uint32_t v = __builtin_amdgcn_perm(hi, lo, ((o) | ((o + 1) << 8)) * 0x00010001u);
    const uint32_t u = __builtin_amdgcn_perm(hi, lo, ((o + 1) | ((o + 2) << 8)) * 0x00010001u);
    p[0] = and_or(v, 0x00380007u, m.a);
    p[1] = and_or(v >> 6, 0x00380007u, m.a);
    p[2] = and_or(u, 0x03800070u, m.b);
    p[3] = and_or(u >> 6, 0x03800070u, m.b);
  }
}

// the MFMA weight operand of step t of the window (t is a constant after unrolling), columns in memory order
template <int BITS, bool BF16, int T, bool WIDE = false>
__device__ __forceinline__ uint4 code_step(const RawCodes<BITS, T>& r, int t, const CodeGroup<BITS, BF16>& g, const CodeMagic& m) {
  typedef CodeForm<BITS, BF16> F;
  uint32_t p[4], d[4];
  code_pairs<BITS, BF16, T>(r, t, m, p);
  if constexpr (BF16) {
    float f[8];
    auto weight = [&](float member, float c) { return WIDE ? (member - c) * g.s : __builtin_fmaf(member, g.s, c); };
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const half2_t h = as_half2(p[j]);
      f[F::kFar ? j : 2 * j] = weight((float)h.x, F::is_b(j) ? g.nblo : g.nalo);
      f[F::kFar ? j + 4 : 2 * j + 1] = weight((float)h.y, F::is_b(j) ? g.nbhi : g.nahi);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) d[j] = pack_bf16(f[2 * j], f[2 * j + 1]);
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) d[j] = as_u32((as_half2(p[j]) - (F::is_b(j) ? g.zb : g.za)) * g.s2);
    if constexpr (F::kFar)
      return make_uint4(__builtin_amdgcn_perm(d[1], d[0], 0x05040100u), __builtin_amdgcn_perm(d[3], d[2], 0x05040100u),
                        __builtin_amdgcn_perm(d[1], d[0], 0x07060302u), __builtin_amdgcn_perm(d[3], d[2], 0x07060302u));
  }
  return make_uint4(d[0], d[1], d[2], d[3]);
}

}  // namespace uniql
