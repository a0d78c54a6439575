// Decode batches (2 .. 32 tokens) on MFMA with loads that write LDS directly and no barrier in the loop: y[M][n_keep] = x[M][k_keep] * W'^T.
//
// A block of eight waves owns R = 16 BF rows and all tokens; the groups of the row are dealt to its waves in contiguous runs.  A wave
// moves the codes and the activations of ITS groups into a ring of its own in LDS (128-bit loads that write LDS directly: no
// registers, no vector instructions), reads them back as matrix operands, unpacks (codes.h) and multiplies.  Nothing in the loop is
// shared between waves, so a wave waits for its own loads only; no column of the activations is fetched twice by a block.  Scales and zero
// points of the whole tile are fetched once at the start (the one barrier before the loop).  The eight partial sums meet in LDS and are
// added in order.
//
// LDS, per wave: L slots of activations [token][chunks of 8 columns], a slot per part (a group up to 16 tokens, half a group from
// 17 on), and slots of codes [row][units of 16 bytes], a slot per group; then per block windows of eight scales and sixteen zero points
// of every row.  Chunks and units of a row are permuted by bank_key (pipe_kernel.h).
#pragma once
#include "pipe_kernel.h"
#include "ring_pick.h"

namespace uniql {

constexpr int kRingWaves = 8;
constexpr int kRingWaveLds = 18 * 1024;   // of a wave's ring; the rest is for scales and zero points

struct RingBatch {
  LinearArgs p[kMaxBatch];
  int first[kMaxBatch];   // first tile of problem i
  int n, tiles;
};

// XT: tokens of a slot (4, 8, 16 or 32; at least M)
template <int XT, int BF, int BITS>
struct RingShape {
  static constexpr int AF = (XT + 15) / 16;
  static constexpr int H = AF > 1 ? 2 : 1, T = 4 / H;      // parts of a group, steps of 32 columns in a part
  static constexpr int CH = 16 / H;                        // chunks of a token in a part
  static constexpr int XPart = XT * CH * 16, XL = XPart / 1024;
  static constexpr int U = BITS;                           // units of a row's group
  static constexpr int WL = (BF * 16 * U + 63) / 64, WSlot = WL * 1024;
  static constexpr int R = 16 * BF;
  // Permutation of the units of a row, so that sixteen rows lie on different banks: 64 and 128 bytes a row need it (a lane's pair of units
  // of 8 bits stays together), 48 do not and 96 share a bank between two rows.
  static __device__ __forceinline__ int code_key(int row) {
    return BITS == 4 ? bank_key(row) >> 2 : BITS == 8 ? bank_key(row) >> 2 << 1 : 0;
  }
  static constexpr bool fits(int l) {
    const int ws = (l + H - 1) / H;
    return l * XPart + ws * WSlot <= kRingWaveLds && l * XL + ws * WL <= 63;
  }
  static constexpr int most() {
    int l = 1;
    while (l < 4 * H && fits(l + 1)) ++l;
    return l;
  }
  static constexpr int L = most(), WS = (L + H - 1) / H;   // slots of activations (parts in flight), of codes
  static constexpr int WaveLds = L * XPart + WS * WSlot;
  static constexpr int Red = kRingWaves * AF * BF * 1024;
  static constexpr bool Valid = fits(1) && Red <= kRingLds;
  // loads of parts q + 1 .. q + r where q % H == p
  static constexpr int loads(int p, int r) {
    int n = 0;
    for (int j = 1; j <= r; ++j) n += XL + ((p + j) % H == 0 ? WL : 0);
    return n;
  }
  static int lds(int ngroups) {
    const int sz = ((ngroups + 7) / 8 + (ngroups + 15) / 16) * R * 16 + 256, ring = kRingWaves * WaveLds + sz;
    return ring > Red ? ring : Red;
  }
};

// A load of 64 x 16 bytes (ring_load_word: 64 x 4) that writes LDS: the wave's active lanes, lane i at lds + 16 i.  (As asm, so that
// the compiler does not make every later LDS read of the wave wait for it: the kernel waits for exactly the loads that it needs.  The
// output is LDS; m0, which the compiler warns of as one of its own, is the only register written.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void ring_load(u32x4_t rsrc, uint32_t lds, int voff, int soff) {
#ifdef __HIP_DEVICE_COMPILE__
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory", "m0");
#endif
}

__device__ __forceinline__ void ring_load_word(u32x4_t rsrc, uint32_t lds, int voff) {
#ifdef __HIP_DEVICE_COMPILE__
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" ::"s"(lds), "v"(voff), "s"(rsrc) : "memory", "m0");
#endif
}

#pragma clang diagnostic pop

__device__ __forceinline__ u32x4_t ring_rsrc(const void* base, int bytes) {
  const uint64_t b = (uint64_t)base;
  u32x4_t r = {(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b), (uint32_t)__builtin_amdgcn_readfirstlane((int)((b >> 32) & 0xffffu)),
               (uint32_t)__builtin_amdgcn_readfirstlane(bytes), kBufferWord3};
  return r;
}

// Waits until part q (q % H == P) has landed; `rem` later parts are on their way, at most MOST of which count.
template <class S, int P, int N>
__device__ __forceinline__ void ring_wait_last(int rem) {
  if constexpr (N >= 0) {
    if (rem == N) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(S::loads(P, N)) : "memory");
    ring_wait_last<S, P, N - 1>(rem);
  }
}
template <class S, int P, int MOST>
__device__ __forceinline__ void ring_wait(int rem) {
  if (__builtin_expect(rem >= MOST, 1)) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(S::loads(P, MOST)) : "memory");
  else ring_wait_last<S, P, MOST - 1>(rem);
}

// GLU: the gate and the up matrix of a gated MLP (Eq. 1; problems 0 and 1: the same activations, sizes and number of kept rows).  Fragments of a block
// are gate rows and up rows of one row tile in turn, and the wave that adds the partial sums of both stores h = SiLU(g) * u, rounded once.
template <int XT, int BF, int BITS, bool BF16, bool SEG, bool GLU>
__global__ __launch_bounds__(kRingWaves * kWave, 2) void w_ring_kernel(RingBatch bt) {
#ifdef __HIP_DEVICE_COMPILE__
  typedef RingShape<XT, BF, BITS> S;
  constexpr int AF = S::AF, H = S::H, T = S::T, CH = S::CH, XL = S::XL, WL = S::WL, U = S::U, L = S::L, R = S::R;
  static_assert(!GLU || (BITS == 4 && BF % 2 == 0 && S::AF == 1 && !SEG), "pairs of fragments");
  constexpr int NM = GLU ? 2 : 1;                          // matrices of a block: fragment b is of matrix b % NM
  extern __shared__ __align__(16) unsigned char smem[];
  typedef __attribute__((address_space(3))) unsigned char lds_byte;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  int pi = 0, tile;
  {
    // a die takes a contiguous stretch of the tiles (neighbours share lines of scales and zero points)
    const int b = (int)blockIdx.x, die = b % kPipeDies, nb = bt.tiles;
    tile = die * (nb / kPipeDies) + (die < nb % kPipeDies ? die : nb % kPipeDies) + b / kPipeDies;
#pragma unroll
    for (int i = 1; i < kMaxBatch; ++i) pi += (i < bt.n && tile >= bt.first[i]) ? 1 : 0;
    tile -= bt.first[pi];
  }
  const LinearArgs a = bt.p[pi];
  const KeepMap& km = a.km;
  const int n0 = tile * (R / NM);
  auto stored = [&](int m, int rc) {                       // compact row of matrix m -> stored row (past the last one: a valid, unused row)
    rc = rc < km.n_keep ? rc : km.n_keep - 1;
    return stored_row(GLU && m == 1 ? bt.p[1].km : km, rc);
  };
  const int row_bytes = a.K_total / 8 * BITS, gpr = a.K_total / kGroup;
  const int ngroups = (km.k_span + kGroup - 1) / kGroup;
  // this wave's groups; the first waves, which lie on different SIMDs, take one more
  const int base = ngroups / kRingWaves, over = ngroups - base * kRingWaves;
  const int ng = base + (wave < over ? 1 : 0), g0 = wave * base + (wave < over ? wave : over);
  const int parts = ng * H;

  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte*)smem;
  const int ring0 = wave * S::WaveLds, wring0 = ring0 + L * S::XPart;
  const int sz0 = kRingWaves * S::WaveLds, nws = (ngroups + 7) / 8, nwz = (ngroups + 15) / 16, zz0 = sz0 + nws * R * 16;
  uint32_t zmask[NM], zdef[NM];                            // (without zero points every one is the middle of the range)

  const u32x4_t rx = ring_rsrc(a.x, (int)(((long long)(a.M - 1) * a.ldx + km.k_keep) * 2));
  u32x4_t rw[NM];
#pragma unroll
  for (int m = 0; m < NM; ++m) {
    const LinearArgs& w = bt.p[GLU ? m : pi];
    rw[m] = ring_rsrc(w.qweight, w.N_total * row_bytes);
    zmask[m] = w.zeros ? 0xffu : 0u, zdef[m] = w.zeros ? 0u : 1u << (BITS - 1);
  }

  // ---- an odd last column of a prefix, whose word may lie partly past the resource and then reads as zero (see clear, below): from the
  // word that ends with it, a lane per token
  const int tail = SEG ? 0 : km.k_keep & 7;
  const int odd0 = zz0 + nwz * R * 16;
  if ((tail & 1) && ng > 0 && g0 + ng == ngroups && lane < a.M) ring_load_word(rx, lds0 + odd0, lane * (int)a.ldx * 2 + (km.k_keep - 2) * 2);

  // ---- scales and zero points: window w of eight (sixteen) groups of every row of the tile, windows dealt to the waves.  A window never
  // leaves the row (at the row's end it starts earlier); but that of the zero points of a row of fewer than sixteen groups ends in the next row, and the
  // last row's, whose last word could lie partly past the array, starts earlier and is moved in LDS (below).
  {
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const LinearArgs& w = bt.p[GLU ? m : pi];
      const u32x4_t rs = ring_rsrc(w.scales, w.N_total * gpr * 2);
      const u32x4_t rz = ring_rsrc(w.zeros, w.zeros ? w.N_total * gpr : 0);
      const int zlast = gpr < 16 ? w.N_total * gpr - 16 : (w.N_total - 1) * gpr;   // where the last row's window starts
#pragma unroll
      for (int p = 0; p < (R + 63) / 64; ++p) {
        const int r = p * 64 + lane, e0 = stored(m, GLU ? n0 + (r >> 5) * 16 + (r & 15) : n0 + r) * gpr;
        if (r < R && (!GLU || (r >> 4 & 1) == m)) {
          for (int i = wave; i < nws; i += kRingWaves)
            ring_load(rs, lds0 + sz0 + (i * R + p * 64) * 16, 2 * e0, 2 * (8 * i < gpr - 8 ? 8 * i : gpr - 8));
          if (w.zeros)
            for (int i = kRingWaves - 1 - wave; i < nwz; i += kRingWaves)
              ring_load(rz, lds0 + zz0 + (i * R + p * 64) * 16, e0 < zlast ? e0 : zlast, gpr < 16 || 16 * i < gpr - 16 ? 16 * i : gpr - 16);
        }
      }
    }
  }

  // ---- where this lane's units of a part lie.  Segments divide the groups, so every group is alike: its kept columns are `kpg`
  // consecutive ones of x.
  const int seg_shift = SEG ? __builtin_ctz((unsigned)km.cs_stride) : 0;
  const int kpg = SEG ? (kGroup >> seg_shift) * km.cs_keep : kGroup, ldx2 = (int)a.ldx * 2;
  auto key = [](int tok) { return H == 2 ? bank_key(tok) >> 1 : bank_key(tok); };
  auto unit = [&](int k, int p, int kept) {     // kept: columns of the group that a prefix keeps
    const int v = k * 64 + lane, tok = v / CH, c = (v % CH) ^ key(tok), k0 = (p * CH + c) * 8;
    int col = k0;
    bool there = k0 < kept;
    if constexpr (SEG) {
      const int off = k0 & (km.cs_stride - 1);
      col = (k0 >> seg_shift) * km.cs_keep + off;
      there = off < km.cs_keep;
    }
    return there ? tok * ldx2 + col * 2 : kBeyond;
  };
  int xoff[SEG ? H : 1][XL], woff[WL];
#pragma unroll
  for (int p = 0; p < (SEG ? H : 1); ++p)
#pragma unroll
    for (int k = 0; k < XL; ++k) xoff[p][k] = unit(k, p, kGroup);
#pragma unroll
  for (int k = 0; k < WL; ++k) {
    const int v = k * 64 + lane, row = v / U, j = v - row * U, js = j ^ S::code_key(row);
    woff[k] = stored(k % NM, GLU ? n0 + (row >> 5) * 16 + (row & 15) : n0 + row) * row_bytes + js * 16;   // (GLU: a load is a fragment)
    if ((R * U) % 64 != 0 && row >= R) woff[k] = kBeyond;  // (the last load's lanes behind the tile)
  }
  const int whole = SEG ? ngroups : km.k_keep / kGroup;    // groups that are kept as a whole
  // part p of the wave's group i, into slots xs and ws
  auto issue = [&](int i, int p, int xs, int ws) {
    const int g = g0 + i;
    if (p == 0) {
#pragma unroll
      for (int k = 0; k < WL; ++k) ring_load(rw[k % NM], lds0 + wring0 + ws * S::WSlot + k * 1024, woff[k], g * (U * 16));
    }
    const uint32_t to = lds0 + ring0 + xs * S::XPart;
    if (g < whole) {
#pragma unroll
      for (int k = 0; k < XL; ++k) ring_load(rx, to + k * 1024, xoff[SEG ? p : 0][k], g * (kpg * 2) + (SEG ? 0 : p * (CH * 16)));
    } else {
#pragma unroll
      for (int k = 0; k < XL; ++k) ring_load(rx, to + k * 1024, unit(k, p, km.k_keep - g * kGroup), g * (kpg * 2));
    }
  };
  int issued = 0, xs_in = 0, ws_in = 0;                    // parts, next slots
  auto issue_next = [&]() {
    const int i = issued / H, p = issued % H;
    if (H == 1 || p == 0) issue(i, 0, xs_in, ws_in);
    else issue(i, 1, xs_in, ws_in);
    xs_in = xs_in + 1 == L ? 0 : xs_in + 1;
    if (p == H - 1) ws_in = ws_in + 1 == S::WS ? 0 : ws_in + 1;
    ++issued;
  };
#pragma unroll
  for (int q = 0; q < L; ++q)
    if (q < parts) issue_next();

  // ---- operands: activations of step t, codes of the group's row, constants
  const int n = lane & 15, ks = lane >> 4;
  const int tok = XT < 16 ? n & (XT - 1) : n;
  int xrd[T], wrd[H];
#pragma unroll
  for (int t = 0; t < T; ++t) xrd[t] = ring0 + (tok * CH + ((ks * T + t) ^ key(tok))) * 16;
#pragma unroll
  for (int p = 0; p < H; ++p) {
    const int byte = p * (8 * BITS) + (T * BITS % 4 == 0 ? ks * (T * BITS) : 0);   // (windows inside words: read_codes finds them from ks)
    wrd[p] = wring0 + n * (U * 16) + (((byte >> 4) ^ S::code_key(n)) << 4) + (byte & 15);
  }
  float4_t acc[AF][BF];
#pragma unroll
  for (int f = 0; f < AF; ++f)
#pragma unroll
    for (int b = 0; b < BF; ++b) acc[f][b] = float4_t{0.f, 0.f, 0.f, 0.f};
  const CodeMagic mg = make_code_magic<BITS, BF16>();

  // scales and zero points of this wave have landed, then everybody's
  ring_wait<S, H - 1, L>(parts);
  if (!GLU && gpr < 16 && wave == kRingWaves - 1 && a.zeros) {   // (the wave that has loaded the only window)
#pragma unroll
    for (int p = 0; p < (R + 63) / 64; ++p) {
      const int r = p * 64 + lane;
      if (r < R && stored(0, n0 + r) == a.N_total - 1) {
        unsigned __int128* z = reinterpret_cast<unsigned __int128*>(smem + zz0 + r * 16);
        *z >>= 8 * (16 - gpr);
      }
    }
  }
  pipe_barrier();

  // What lies behind the kept columns in a part's last block of a prefix, or in the last blocks of its segments, is cleared: the next
  // segment's first columns, or the next token's.
  auto clear = [&](int g, int p, unsigned char* to) {
    if constexpr (SEG) {
      const int partial = km.cs_keep & 7;
      const int log = seg_shift < (H == 2 ? 6 : 7) ? (H == 2 ? 6 : 7) - seg_shift : 0;     // segments of a part
      for (int i = lane; i < XT << log; i += 64) {
        const int t = i >> log, k0 = ((i & ((1 << log) - 1)) << seg_shift) + (km.cs_keep & ~7);   // in the part (128 columns: in the group)
        const int c = k0 / 8 - (seg_shift == 7 ? p * CH : 0);
        if (c < 0 || c >= CH) continue;
        uint32_t* w = reinterpret_cast<uint32_t*>(to + (t * CH + (c ^ key(t))) * 16);
        if (partial == 2) w[1] = 0u;
        if (partial <= 4) w[2] = 0u;
        w[3] = 0u;
      }
    } else {
      const int c = km.k_keep / 8 - g * 16 - p * CH, keep = tail & ~1;
      if (c < 0 || c >= CH || lane >= XT) return;
      auto m = [&](int i) { return keep > i ? ~0u : 0u; };
      const uint32_t odd = (tail & 1) && lane < a.M ? reinterpret_cast<const uint32_t*>(smem + odd0)[lane] >> 16 : 0u;
      uint4* w = reinterpret_cast<uint4*>(to) + lane * CH + (c ^ key(lane));
      uint4 v = *w;
      v.x = (v.x & m(0)) | (tail == 1 ? odd : 0u);
      v.y = (v.y & m(2)) | (tail == 3 ? odd : 0u);
      v.z = (v.z & m(4)) | (tail == 5 ? odd : 0u);
      v.w = tail == 7 ? odd : 0u;
      *w = v;
    }
  };

  typedef RawCodes<BITS, T> Raw;
  int xs = 0, ws = 0;
  for (int i = 0; i < ng; ++i) {
    const int g = g0 + i;
    Raw raw[H][BF];
    uint32_t sb[BF], zb[BF];
    CodeGroup<BITS, BF16> gq[BF];
    bool wide = false;
#pragma unroll
    for (int p = 0; p < H; ++p) {
      const int rem = parts - 1 - (i * H + p);
      if (p == 0) ring_wait<S, 0, L - 1>(rem);
      else ring_wait<S, H - 1, L - 1>(rem);
      unsigned char* const xp = smem + xs * S::XPart;
      if (SEG ? (km.cs_keep & 7) != 0 : g >= whole && tail != 0) clear(g, p, xp + ring0);
      uint4 av[T][AF];
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int f = 0; f < AF; ++f) av[t][f] = *reinterpret_cast<const uint4*>(xp + xrd[t] + f * (16 * CH * 16));
      if (p == 0) {
        const unsigned char* const wp = smem + ws * S::WSlot;
#pragma unroll
        for (int b = 0; b < BF; ++b)
#pragma unroll
          for (int h = 0; h < H; ++h) raw[h][b] = read_codes<BITS, T>(wp + wrd[h] + b * (16 * U * 16), T * BITS % 4 == 0 ? 0 : ks);
        const int gs = g & ~7, gz = g & ~15;
        const unsigned char* const sp = smem + sz0 + (g >> 3) * (R * 16) + 2 * (g - (gs < gpr - 8 ? gs : gpr - 8)) + n * 16;
        const unsigned char* const zp = smem + zz0 + (g >> 4) * (R * 16) + g - (gpr < 16 || gz < gpr - 16 ? gz : gpr - 16) + n * 16;
#pragma unroll
        for (int b = 0; b < BF; ++b) sb[b] = *reinterpret_cast<const uint16_t*>(sp + b * 256);
#pragma unroll
        for (int b = 0; b < BF; ++b) zb[b] = (zp[b * 256] & zmask[b % NM]) | zdef[b % NM];
        ws = ws + 1 == S::WS ? 0 : ws + 1;
      }
      xs = xs + 1 == L ? 0 : xs + 1;
      // everything of the slot is in registers: the loads that take it may go
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (issued < parts) issue_next();
      auto multiply = [&](auto wide_form) {
        constexpr bool W = decltype(wide_form)::value;
#pragma unroll
        for (int b = 0; b < BF; ++b) {
          if (p == 0) gq[b] = make_code_group<BITS, BF16, W>(sb[b], zb[b]);
#pragma unroll
          for (int t = 0; t < T; ++t) {
            const uint4 wf = code_step<BITS, BF16, T, W>(raw[p][b], t, gq[b], mg);
#pragma unroll
            for (int f = 0; f < AF; ++f) acc[f][b] = mfma_16x16x32<BF16>(wf, av[t][f], acc[f][b]);
          }
        }
      };
      if constexpr (BF16) {
        if (p == 0) {
          uint32_t largest = 0;
#pragma unroll
          for (int b = 0; b < BF; ++b) largest = max(largest, sb[b] << 17);
          wide = __builtin_amdgcn_ballot_w64(largest >= kScaleWide << 17) != 0;
        }
        if (__builtin_expect(wide, 0)) multiply(std::true_type());
        else multiply(std::false_type());
      } else {
        multiply(std::false_type());
      }
    }
  }

  // ---- partial sums through LDS (nobody reads or moves slots any more), fragment q added up in order and stored by wave q % 8
  pipe_barrier();
  float4_t* red = reinterpret_cast<float4_t*>(smem);
#pragma unroll
  for (int f = 0; f < AF; ++f)
#pragma unroll
    for (int b = 0; b < BF; ++b) red[(wave * AF * BF + f * BF + b) * 64 + lane] = acc[f][b];
  pipe_barrier();
  for (int q = wave; q < AF * BF / NM; q += kRingWaves) {
    float4_t s = red[q * NM * 64 + lane];
#pragma unroll
    for (int k = 1; k < kRingWaves; ++k) s += red[(k * AF * BF + q * NM) * 64 + lane];
    if constexpr (GLU) {
      float4_t u = red[(q * 2 + 1) * 64 + lane];
#pragma unroll
      for (int k = 1; k < kRingWaves; ++k) u += red[(k * AF * BF + q * 2 + 1) * 64 + lane];
#pragma unroll
      for (int v = 0; v < 4; ++v) s[v] = s[v] * u[v] * __builtin_amdgcn_rcpf(1.0f + __expf(-s[v]));
    }
    // lane l holds token l % 16 of the fragment, rows 4 (l / 16) + v
    const int f = q / (BF / NM), b = q - f * (BF / NM), to = f * 16 + n, rc = n0 + b * 16 + 4 * ks;
    if (to >= a.M || rc >= km.n_keep) continue;
    half_t* y = a.y + (size_t)to * a.ldy + rc;
    uint16_t o[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) o[v] = __builtin_bit_cast(uint16_t, out16<BF16>(s[v]));
    if (rc + 4 <= km.n_keep) {
      typedef uint32_t u32x2_u2 __attribute__((ext_vector_type(2), aligned(2)));
      u32x2_u2 pk;
      pk.x = o[0] | ((uint32_t)o[1] << 16);
      pk.y = o[2] | ((uint32_t)o[3] << 16);
      *reinterpret_cast<u32x2_u2*>(y) = pk;
    } else {
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (rc + v < km.n_keep) y[v] = __builtin_bit_cast(half_t, o[v]);
    }
  }
#endif
}

template <int XT, int BF, int BITS, bool BF16, bool SEG, bool GLU = false>
static hipError_t ring_launch(const LinearArgs* p, int n, hipStream_t stream) {
  typedef RingShape<XT, BF, BITS> S;
  if constexpr (!S::Valid) {
    return hipErrorInvalidValue;
  } else {
    auto kern = w_ring_kernel<XT, BF, BITS, BF16, SEG, GLU>;
    RingBatch b;
    b.n = n;
    int tiles = 0, most = 0;
    for (int i = 0; i < kMaxBatch; ++i) {
      b.p[i] = p[i < n ? i : 0];
      b.first[i] = tiles;
      if (i >= n) continue;
      if (!GLU) tiles += (p[i].km.n_keep + S::R - 1) / S::R;
      else tiles = (p[i].km.n_keep + S::R / 2 - 1) / (S::R / 2);
      const int ng = (p[i].km.k_span + kGroup - 1) / kGroup;
      most = ng > most ? ng : most;
    }
    if (GLU) b.n = 1;                                      // (tiles are those of the pair)
    b.tiles = tiles;
    const int lds = S::lds(most);
    if (lds > kRingLds) return hipErrorInvalidValue;
    // (the limit is the kernel's, not the launch's: the same from every thread, or one could lower it between another's set and launch)
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kRingLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(tiles), dim3(kRingWaves * kWave), lds, stream, b);
    return hipGetLastError();
  }
}

}  // namespace uniql
