// W4A16 GEMM on MFMA for M >= 2 tokens: y[M][n_keep] = x[M][k_keep] * W'^T.
//
// "Direct-B" design: the packed weights never pass through LDS.  With
// v_mfma_f32_16x16x32_f16 the weight operand of lane l is 8 consecutive input columns of
// output row (l % 16) in k-slot (l / 16), which is exactly one 32-bit word of packed codes, so a
// wave fetches its 16 rows x 128 columns (one quantisation group per row) with ONE 128-bit load
// per lane (word t of the load feeds MFMA t of the group) and dequantises in registers to the
// canonical fp16 weights.  Only the activations go through LDS: the block stages a slab of x
// (its tokens x the columns of the current step) at *stored* column positions, zeros where
// pruned, pre-permuted inside every 8-column block to the (0,4,1,5,2,6,3,7) order the unpack
// produces, double-buffered so that the next slab is fetched while the current one is used.
//
// A wave owns BF fragments of 16 rows and AF fragments of 16 tokens (AF*BF accumulators of 4
// VGPRs); a dequantised weight fragment is reused by AF MFMAs, an activation fragment by BF.
// It serves the prompts whose tiles of 128 or 64 tokens x 256 rows fill the chip better than those of the
// pipelined kernel (pipe_kernel.h), and every column rule and size the other kernels do not take: up to 64 tokens with
// the K range split over KS waves of the block (reduced through LDS at the end).
#pragma once
#define UNIQL_ANDOR_PLAIN   // and-or as plain C here: the scheduler must be able to classify it as VALU
#include "common.h"
#include "smallm_kernel.h"
#include "prefill_kernel.h"
#include "pipe_dispatch.h"
#include "ring_pick.h"
#include <type_traits>

namespace uniql {

struct WTile {
  uint4 w;
};

// AF token fragments, BF row fragments per wave, WN waves along rows, KS waves along K,
// S2 groups per wave and iteration (the slab holds KS * S2 groups: fewer, longer iterations hide
// the latency of fetching the next slab), PW iterations of weight loads kept in flight.
// BF16: scales, x and y are bfloat16; the weights are rounded to bfloat16 and the MFMA is the bf16 one.
template <int AF, int BF, int WN, int KS, int S2, int PW, int XM, bool BF16>
__global__ __launch_bounds__(WN * KS * 64) void w4_mfma_kernel(LinearArgs a) {
  // activation staging mode: 0 = element by element through the column map, 1 = column prefix,
  // 2 = column segments whose stride is a multiple of 8 (128-bit loads in both)
  constexpr bool XVEC = XM == 1, XSEG = XM == 2;
  constexpr int NT = WN * KS * 64;
  constexpr int BM = 16 * AF;               // tokens per block
  constexpr int BN = WN * BF * 16;          // rows per block
  constexpr int SC = KS * S2 * 128;         // columns per slab (S2 groups per K-split wave)
  constexpr int NCH = SC / 8;               // 8-column chunks per slab
  constexpr int UNITS = BM * NCH;           // 16-byte units per slab
  static_assert(UNITS % NT == 0, "slab must divide evenly over the threads");
  constexpr int UPT = UNITS / NT;           // units per thread

  extern __shared__ __align__(16) unsigned char smem[];
  // Slab layout [2][NCH][BM] of 16-byte units (8 columns of one token).  The 16 lanes that read one
  // activation fragment (16 tokens, one chunk) touch one aligned 256-byte window, which is what
  // ds_read_b128 needs to run at the full LDS rate on this target (a padded token-major slab reads
  // at half rate).  Inside its window token j sits at slot j ^ swz(chunk), swz = (k-slot | step << 2)
  // of the chunk, so that the 16 lanes that WRITE 16 consecutive chunks of one token also hit 16
  // different bank groups; measured, both patterns are conflict-free.
  uint4* xs = reinterpret_cast<uint4*>(smem);
  // Scales and zero points of the slab's groups ride along: [2][BN][KS * S2] words (scale bits |
  // zero << 16).  A load whose lanes touch 16 different rows costs the memory pipeline about 4
  // clocks per row whatever its width, so instead of every wave fetching the two values of its 16
  // rows per group, one thread per (row, group) of the block fetches them with the slab, adjacent
  // lanes reading adjacent groups of a row.
  constexpr int NG = KS * S2;                // groups per slab
  static_assert(BN * NG <= NT, "one thread per (row, group) of a slab");
  uint32_t* szs = reinterpret_cast<uint32_t*>(smem + (size_t)2 * UNITS * sizeof(uint4));

  const KeepMap& km = a.km;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wn = wave % WN, wk = wave / WN;
  const int n = lane & 15, ks = lane >> 4;
  // Block -> tile.  Consecutive blocks of a launch go to the eight dies (XCDs) in turn, each with an L2 of its own, so
  // block b runs on die b % 8.  Blocks are renumbered so that a die's blocks are consecutive tiles of a walk that
  // takes kTokTilesPerPass token tiles at a time and, inside that, row tile by row tile: the 32 blocks a die runs at
  // once then cover 8 row tiles x 4 token tiles and share their weight rows and activation slabs through that die's
  // L2 (with the launch order, a token tile's activations were fetched once per die: 857 MB of L2 misses for the
  // 159 MB of the 4096-token down projection).
  int rt = blockIdx.x, tt = blockIdx.y;
  if (gridDim.y > 1) {
    constexpr int kDies = 8, kTokTilesPerPass = 4;
    const int nrt = gridDim.x, ntt = gridDim.y, nb = nrt * ntt;
    const int bid = blockIdx.y * nrt + blockIdx.x;
    const int die = bid % kDies, j = bid / kDies;
    const int L = die * (nb / kDies) + min(die, nb % kDies) + j;   // blocks of die 0, then of die 1, ...
    const int full = (ntt / kTokTilesPerPass) * kTokTilesPerPass;  // token tiles in whole passes
    const int in_full = nrt * full;
    if (L < in_full) {
      const int pass = L / (nrt * kTokTilesPerPass), r = L - pass * (nrt * kTokTilesPerPass);
      rt = r / kTokTilesPerPass;
      tt = pass * kTokTilesPerPass + (r - rt * kTokTilesPerPass);
    } else {
      const int w = ntt - full, r = L - in_full;                   // the last, narrower pass
      rt = r / w;
      tt = full + (r - rt * w);
    }
  }
  const int n0 = rt * BN, m0 = tt * BM;
  const int words_per_row = a.K_total >> 3, groups_per_row = a.K_total / kGroup;
  const int ngroups = (km.k_span + kGroup - 1) / kGroup;
  const int nit = (ngroups + KS * S2 - 1) / (KS * S2);
  const int nit_pw = (nit + PW - 1) / PW * PW;   // loop trip count; extra iterations multiply zeros

  // stored row of each of this lane's weight fragments (clamped: every address stays valid)
  size_t wrow[BF];
#pragma unroll
  for (int bf = 0; bf < BF; ++bf) {
    int rc = n0 + (wn * BF + bf) * 16 + n;
    rc = rc < km.n_keep ? rc : km.n_keep - 1;
    wrow[bf] = (size_t)stored_row(km, rc);
  }
  // group s2 of iteration it for this wave: slab-local group s2 * KS + wk
  auto load_w = [&](int it, WTile (&t)[S2][BF]) {
#pragma unroll
    for (int s2 = 0; s2 < S2; ++s2) {
      int g = (it * S2 + s2) * KS + wk;
      g = g < ngroups ? g : ngroups - 1;   // past the end: a valid, redundant load (x is zero there)
#pragma unroll
      for (int bf = 0; bf < BF; ++bf)
        t[s2][bf].w = *reinterpret_cast<const uint4*>(a.qweight + wrow[bf] * words_per_row + g * 16 + ks * 4);
    }
  };
  // this thread's (row, group) of the scale / zero staging, if it has one
  const bool sz_owner = tid < BN * NG;
  size_t sz_row;
  {
    int rc = n0 + tid / NG;
    rc = rc < km.n_keep ? rc : km.n_keep - 1;
    sz_row = (size_t)stored_row(km, rc) * groups_per_row;
  }
  auto fetch_sz = [&](int it, uint32_t& sbits, uint32_t& z) {
    int g = it * NG + tid % NG;
    g = g < ngroups ? g : ngroups - 1;
    sbits = a.scales[sz_row + g];
    z = a.zeros ? a.zeros[sz_row + g] : 8u;   // no zero points: the symmetric scheme, z = 8
  };

  // x slab staging: unit u of a slab = token (u / NCH), 8-column chunk (u % NCH).
  // fetch_x only issues loads (unconditional, on clamped addresses) and records which halves are
  // real; store_x, one iteration later, masks, permutes and writes them to LDS.  Nothing touches
  // the loaded registers in between, so the wave never waits for x at the point of issue.
  // XVEC: whole 8-column blocks below kv come from one 128-bit load; the up to 7 kept columns at
  // and after kv are added in the epilogue.  XSEG: a block lies in one segment and its kept columns
  // are its first nk, contiguous in x: one 128-bit load and a per-half mask (only the block that
  // holds a row's last kept columns, fewer than 8 of them, is read element by element).
  // Otherwise: eight element loads through the column map.
  auto unit_token = [](int u) { return u / NCH; };
  auto unit_chunk = [](int u) { return u % NCH; };
  auto swz = [](int chunk) { return ((chunk >> 2) & 3) | ((chunk & 3) << 2); };
  const int kv = km.k_keep & ~7;
  const uint16_t* xbits = reinterpret_cast<const uint16_t*>(a.x);
  struct XRegs {
    uint4 v[XM != 0 ? UPT : 1];
    uint32_t e[XM != 0 ? 1 : UPT][8];
    uint32_t ok[UPT];   // XVEC: all-ones / zero word mask; otherwise bit j = half j is real
  };
  auto fetch_x = [&](int it, XRegs& xr) {
#pragma unroll
    for (int i = 0; i < UPT; ++i) {
      const int u = tid + i * NT;
      const int tk = unit_token(u), cb = unit_chunk(u);
      const int k0 = it * SC + cb * 8;
      const int tok = m0 + tk;
      const bool tok_ok = tok < a.M;
      const size_t xoff = (size_t)(tok_ok ? tok : a.M - 1) * a.ldx;
      if constexpr (XVEC) {
        const bool full = k0 + 8 <= kv;
        xr.v[i] = load_u4_unaligned(a.x + xoff + (full ? k0 : 0));
        xr.ok[i] = (full && tok_ok) ? 0xffffffffu : 0u;
      } else if constexpr (XSEG) {
        const int seg = k0 / km.cs_stride, off = k0 - seg * km.cs_stride;
        int nk = km.cs_keep - off;                       // kept columns at the start of this block
        nk = nk < 0 ? 0 : (nk > 8 ? 8 : nk);
        nk = k0 < km.k_span ? nk : 0;
        const int c = seg * km.cs_keep + off;            // compact column of the block's first column
        const bool vec = nk > 0 && c + 8 <= km.k_keep;   // the 16 bytes at c lie inside the token row
        xr.v[i] = load_u4_unaligned(a.x + xoff + (vec ? c : 0));
        xr.ok[i] = tok_ok ? (1u << nk) - 1u : 0u;
        if (nk > 0 && !vec) {   // the row's last kept columns, fewer than 8 left
          uint32_t h[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) h[j] = j < nk ? (uint32_t)xbits[xoff + c + j] : 0u;
          xr.v[i] = make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16));
        }
      } else {
        xr.ok[i] = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int k = k0 + j;
          const int kc = k < km.k_span ? compact_col(km, k) : -1;
          xr.e[i][j] = xbits[xoff + (kc >= 0 ? kc : 0)];
          xr.ok[i] |= (kc >= 0 && tok_ok) ? (1u << j) : 0u;
        }
      }
    }
  };
  // registers -> LDS: the unit's 8 halves in the pair order of the unpack, (0,4) (1,5) (2,6) (3,7): with 128-bit loads
  // a mask per loaded word, then one byte permute per output word
  auto store_x = [&](int buf, const XRegs& xr) {
#pragma unroll
    for (int i = 0; i < UPT; ++i) {
      const int u = tid + i * NT;
      const int tk = unit_token(u), cb = unit_chunk(u);
      uint4 o;
      if constexpr (XVEC || XSEG) {
        uint4 r = xr.v[i];
        if constexpr (XVEC) {
          const uint32_t m = xr.ok[i];
          r.x &= m; r.y &= m; r.z &= m; r.w &= m;
        } else {
          // kept columns are the unit's first nk: a mask per 32-bit word (halves 2 w and 2 w + 1)
          const uint32_t ok = xr.ok[i];
          r.x &= (ok & 1u ? 0xffffu : 0u) | (ok & 2u ? 0xffff0000u : 0u);
          r.y &= (ok & 4u ? 0xffffu : 0u) | (ok & 8u ? 0xffff0000u : 0u);
          r.z &= (ok & 16u ? 0xffffu : 0u) | (ok & 32u ? 0xffff0000u : 0u);
          r.w &= (ok & 64u ? 0xffffu : 0u) | (ok & 128u ? 0xffff0000u : 0u);
        }
        o = make_uint4(__builtin_amdgcn_perm(r.z, r.x, 0x05040100u), __builtin_amdgcn_perm(r.z, r.x, 0x07060302u),
                       __builtin_amdgcn_perm(r.w, r.y, 0x05040100u), __builtin_amdgcn_perm(r.w, r.y, 0x07060302u));
      } else {
        uint32_t e[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) e[j] = (xr.ok[i] >> j) & 1u ? xr.e[i][j] : 0u;
        o = make_uint4(e[0] | (e[4] << 16), e[1] | (e[5] << 16), e[2] | (e[6] << 16), e[3] | (e[7] << 16));
      }
      xs[(buf * NCH + cb) * BM + (tk ^ swz(cb))] = o;
    }
  };

  float4_t acc[AF][BF];
#pragma unroll
  for (int af = 0; af < AF; ++af)
#pragma unroll
    for (int bf = 0; bf < BF; ++bf) acc[af][bf] = float4_t{0.f, 0.f, 0.f, 0.f};

  const Magic mg = make_magic();
  WTile ring[PW][S2][BF];
  XRegs xr;
  uint32_t sz_s = 0, sz_z = 0;
#pragma unroll
  for (int p = 0; p < PW; ++p) load_w(p, ring[p]);
  fetch_x(0, xr);
  if (sz_owner) fetch_sz(0, sz_s, sz_z);
  store_x(0, xr);
  if (sz_owner) szs[tid] = sz_s | (sz_z << 16);
  __syncthreads();

  for (int it0 = 0; it0 < nit_pw; it0 += PW) {
#pragma unroll
    for (int p = 0; p < PW; ++p) {
      const int it = it0 + p;
      const int buf = it & 1;
      // this slab's scales and zero points, read before anything else so that the LDS latency is
      // covered by issuing the loads below
      uint32_t szv[S2][BF];
#pragma unroll
      for (int s2 = 0; s2 < S2; ++s2)
#pragma unroll
        for (int bf = 0; bf < BF; ++bf) szv[s2][bf] = szs[(buf * BN + (wn * BF + bf) * 16 + n) * NG + s2 * KS + wk];
      // fetch the next slab into registers while this one is consumed
      if (it + 1 < nit_pw) fetch_x(it + 1, xr);
      if (sz_owner) fetch_sz(it + 1, sz_s, sz_z);

      // Word t of a lane's 128-bit load feeds MFMA t of the group.  Dequantising word t of every
      // row fragment right before its MFMAs keeps only BF operand fragments live and lets the
      // VALU work of step t+1 issue while the matrix pipe is busy with step t.
#pragma unroll
      for (int s2 = 0; s2 < S2; ++s2) {
        typename GroupOf<BF16>::type gq[BF];
        uint32_t wv[BF][4];
#pragma unroll
        for (int bf = 0; bf < BF; ++bf) {
          const WTile& wt = ring[p][s2][bf];
          gq[bf] = make_group<BF16>(szv[s2][bf] & 0xffffu, szv[s2][bf] >> 16);
          wv[bf][0] = wt.w.x; wv[bf][1] = wt.w.y; wv[bf][2] = wt.w.z; wv[bf][3] = wt.w.w;
        }
        const uint4* xb = xs + (buf * NCH + (s2 * KS + wk) * 16 + ks * 4) * BM;
        // Two-stage pipeline over the group's four MFMA steps: while step t multiplies, the
        // activation fragments of step t+1 are read from LDS and its weights dequantised.
        uint4 av[2][AF], bfrag[2][BF];
        auto stage = [&](int t, uint4 (&ao)[AF], uint4 (&bo)[BF]) {
#pragma unroll
          for (int af = 0; af < AF; ++af) ao[af] = xb[t * BM + af * 16 + (n ^ (ks | (t << 2)))];
#pragma unroll
          for (int bf = 0; bf < BF; ++bf) bo[bf] = dequant_word4<BF16>(wv[bf][t], gq[bf], mg);
        };
        stage(0, av[0], bfrag[0]);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          if (t < 3) stage(t + 1, av[(t + 1) & 1], bfrag[(t + 1) & 1]);
#pragma unroll
          for (int af = 0; af < AF; ++af)
#pragma unroll
            for (int bf = 0; bf < BF; ++bf)
              acc[af][bf] = mfma_16x16x32<BF16>(av[t & 1][af], bfrag[t & 1][bf], acc[af][bf]);
        }
      }
      load_w(it + PW, ring[p]);   // refill the ring slot (clamped past the end)
      if (it + 1 < nit_pw) store_x(buf ^ 1, xr);
      if (sz_owner) szs[(buf ^ 1) * BN * NG + tid] = sz_s | (sz_z << 16);
      __syncthreads();
    }
  }

  // ---- epilogue.  Lane l holds, for fragment (af, bf): row (l % 16), tokens 4 * (l / 16) + v.
  if constexpr (KS > 1) {
    float* red = reinterpret_cast<float*>(smem);   // [KS][WN][AF][BF][4][64], reuses the slab space
    constexpr int PER_WAVE = AF * BF * 4 * 64;
    float* mine = red + (size_t)(wk * WN + wn) * PER_WAVE;
#pragma unroll
    for (int af = 0; af < AF; ++af)
#pragma unroll
      for (int bf = 0; bf < BF; ++bf)
#pragma unroll
        for (int v = 0; v < 4; ++v) mine[((af * BF + bf) * 4 + v) * 64 + lane] = acc[af][bf][v];
    __syncthreads();
    if (wk != 0) return;
#pragma unroll
    for (int k2 = 1; k2 < KS; ++k2) {
      const float* other = red + (size_t)(k2 * WN + wn) * PER_WAVE;
#pragma unroll
      for (int af = 0; af < AF; ++af)
#pragma unroll
        for (int bf = 0; bf < BF; ++bf)
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[af][bf][v] += other[((af * BF + bf) * 4 + v) * 64 + lane];
    }
  }
  if constexpr (XVEC) {
    // the kept columns kv .. k_keep-1 (fewer than 8: one word of one group per row), in fp32
    if (kv < km.k_keep) {
#pragma unroll
      for (int bf = 0; bf < BF; ++bf) {
        const uint32_t word = a.qweight[wrow[bf] * words_per_row + (kv >> 3)];
        const size_t gi = wrow[bf] * groups_per_row + (kv >> 7);
        const float sf = in16<BF16>(__builtin_bit_cast(half_t, a.scales[gi]));
        const int z = a.zeros ? a.zeros[gi] : 8;
        for (int j = 0; kv + j < km.k_keep; ++j) {
          const int q = (int)((word >> (4 * j)) & 15u);
          const float w = in16<BF16>(out16<BF16>((float)(q - z) * sf));   // the canonical 16-bit weight
#pragma unroll
          for (int af = 0; af < AF; ++af)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const int tok = m0 + af * 16 + 4 * ks + v;
              const float xv = in16<BF16>(a.x[(size_t)(tok < a.M ? tok : a.M - 1) * a.ldx + kv + j]);
              acc[af][bf][v] = __builtin_fmaf(xv, w, acc[af][bf][v]);
            }
        }
      }
    }
  }
#pragma unroll
  for (int af = 0; af < AF; ++af)
#pragma unroll
    for (int bf = 0; bf < BF; ++bf) {
      const int rc = n0 + (wn * BF + bf) * 16 + n;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int tok = m0 + af * 16 + 4 * ks + v;
        if (tok < a.M && rc < km.n_keep) a.y[(size_t)tok * a.ldy + rc] = out16<BF16>(acc[af][bf][v]);
      }
    }
}


template <bool BF16, int AF, int BF, int WN, int KS, int S2, int PW, int XVEC>
static hipError_t launch_cfg(const LinearArgs& a, hipStream_t stream) {
  constexpr int BM = 16 * AF, BN = WN * BF * 16, SC = KS * S2 * 128;
  size_t smem = (size_t)2 * BM * SC * sizeof(half_t) + (size_t)2 * BN * KS * S2 * sizeof(uint32_t);
  const size_t red = KS > 1 ? (size_t)KS * WN * AF * BF * 4 * 64 * sizeof(float) : 0;
  if (red > smem) smem = red;
  auto kern = w4_mfma_kernel<AF, BF, WN, KS, S2, PW, XVEC, BF16>;
  if (smem > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
  }
  dim3 grid((a.km.n_keep + BN - 1) / BN, (a.M + BM - 1) / BM);
  hipLaunchKernelGGL(kern, grid, dim3(WN * KS * 64), smem, stream, a);
  return hipGetLastError();
}

template <bool BF16>
static hipError_t launch_pipe4(const LinearArgs* p, int n, hipStream_t stream) {
  if constexpr (BF16) return launch_pipe_w4_bf16(p, n, stream);
  else return launch_pipe_w4(p, n, stream);
}

template <bool BF16>
static hipError_t launch_ring4(const LinearArgs* p, int n, hipStream_t stream) {
  if constexpr (BF16) return launch_ring_w4_bf16(p, n, stream);
  else return launch_ring_w4(p, n, stream);
}

// gate and up of a decode batch in one launch: what smallm_glu serves.  From 9 tokens on, with rows of sixteen groups and more, the ring
// kernel's form of it: a block stages its activations once for both matrices and every wave loads for itself (12185 x 4096 at 9 and 16 tokens 25.0 -> 18.4 and 28.4 -> 19.8 us, 14208 x 3584 25.7 -> 20.5 and 24.2 -> 21.5,
// 18944 x 3584 36.6 -> 29.8 and 35.2 -> 30.3, 24000 x 4096 41.2 -> 35.2 and 38.5 -> 35.9; 32000 x 4096 43.2 for 48.4).  Up to 8 tokens as the pair
// of linears: not faster.
template <bool BF16>
static hipError_t glu_batch(const LinearArgs* p, hipStream_t stream, bool* done) {
  if (!smallm_glu_serves(p)) {
    *done = false;
    return hipSuccess;
  }
  if (p[0].M >= 9 && (p[0].km.n_keep + 15) / 16 <= kRingTallest && ring_serves(p[0]) && ring_serves(p[1]) && p[0].km.k_span > 15 * kGroup) {
    *done = true;
    if constexpr (BF16) return launch_ring_glu_bf16(p, stream);
    else return launch_ring_glu(p, stream);
  }
  return smallm_glu<BF16>(p, stream, done);
}

// Which kernel a linear of 2 tokens and more takes.  It follows from the linear alone.  kTile*: w4_mfma_kernel with tiles of
// that many tokens x rows, K over that many waves of a block.
enum GemmRoute {
  kSmallM, kRing, kPipe, kPrefill256, kTile128x256, kTile64x256, kTile64x128k2, kTile32x128k2,
  kTile16x16k8, kTile16x64k4, kTile32x16k8, kTile32x64k4, kTile64x32k4, kTile64x64k4
};

// Column segments of 17..32 tokens that the block-staged kernel keeps, before the pipelined one and, with longer rows, before the ring kernel (ring_takes): those
// whose kept columns are not whole blocks of eight, which the pipelined kernel's movers clear slab after slab, in long rows of up to 256 row tiles (more are two rounds
// of the other kernel's waves: 5120 x 8192 23.3 us there, 16.6 here).  24 tokens, there against here, fp16: 98..108 of 128 or 54 of 64 columns
// 1024 x 14208 20.6 / 23.6, 3584 x 8192 16.6 / 16.6, 3584 x 14208 23.2 / 25.2; 26 of 32 columns 1024 x 8192 14.1 / 17.9.  bfloat16, whose
// unpack is longer there, 54 of 64 1024 x 14208 21.5 / 20.6; 26 of 32 1024 x 8192 14.8 / 16.8.
static inline bool segments_stay(const LinearArgs& a) {
  const KeepMap& km = a.km;
  if (km.cs_keep % 8 == 0 || km.n_keep > 4096) return false;
  if (km.cs_stride < 64) return km.k_span > 3400 + km.n_keep / 10;
  return !a.bf16 && km.k_span > 4096 + (km.n_keep > 1024 ? (km.n_keep - 1024) * 3 / 2 : 0);
}

// xm: staging mode of the activations (0 element by element, 1 column prefix, 2 column segments of whole 8-column units)
static inline GemmRoute gemm_route(const LinearArgs& a, int xm) {
  const int row_tiles = (a.km.n_keep + 15) / 16;
  const bool pipe = xm != 0 && pipe_serves(a);
  if (xm != 0 && ring_takes(a, segments_stay(a))) return kRing;
  // What the ring kernel leaves of the decode batches (M <= 32): up to 8 tokens most prefixes of 640 row tiles and more, segments of more row tiles than it takes,
  // rows of fewer than eight groups, from 9 tokens on long rows of 400 row tiles and more.  They are bound by the weight stream and have another kernel of
  // their own (smallm_kernel.h), except tall matrices from 9 tokens on whose activations it cannot stage once per block: a wave that stages its own 16 x 128
  // activations per group costs more than the pipelined kernel's slabs (before the ring kernel 9472 x 4096 at 12 / 24 tokens 16.9 / 23.3 us there,
  // 11.4 / 14.1 here).  A set of such a matrix and short ones, which are the ring kernel's, is two launches: 8192 + 1024 + 1024 rows x 8192 columns at 9 / 24 tokens
  // 21.7 / 27.5 us, 25.4 / 35.3 in one of the block-staged kernel.  Column segments, whose activations a wave of the pipelined kernel gathers for itself, come here
  // from 17 tokens on (but see segments_stay); at 9..16 tokens the two are level.
  const bool tall = row_tiles >= 400 && a.M >= 9 && !(xm == 1 && smallm_pre(a));
  if (smallm_takes(a, xm == 1) && !(pipe && (tall || (xm == 2 && a.M >= 17 && !segments_stay(a))))) return kSmallM;
  if (pipe && a.M <= 64) return kPipe;
  // What neither takes (rows of fewer than eight groups; above the decode batches, or on tall matrices from 9 tokens on,
  // segments that are not a power of two up to a group with an even number kept): K over four or eight waves of a block, or
  // a matrix of a few thousand rows leaves most of the chip idle (4096 x 4096, segments of 256, 48 tokens: 19.5 us; 32 x 128
  // tiles with K over two waves 21.7); tall matrices 64 rows per block (12288 x 896 at 8 tokens 6.4 us; 16 rows 11.4).
  if (a.M <= 16) return row_tiles >= 600 ? kTile16x64k4 : kTile16x16k8;
  if (a.M <= 32) return row_tiles >= 600 ? kTile32x64k4 : kTile32x16k8;
  if (a.M <= 64) return row_tiles >= 600 ? kTile64x64k4 : kTile64x32k4;
  // More tokens: the cheapest of the tiles (launch_cost).  `tail`: what every kept column behind the last whole block of eight
  // costs a round of these tiles, which add such columns up in the epilogue (the pipelined kernel does not: 2560 x 1999 at 2048
  // tokens 65 us in 128 x 256 tiles, 39 there).
  // (Activations staged element by element, xm = 0, take the table of prefixes: prefixes of 5 columns and segments of 7 at 80..2048
  // tokens are at most 4 % slower than with the tiles that 192 blocks and more chose.)
  const float ng = (float)((a.km.k_span + kGroup - 1) / kGroup);
  const int odd_columns = xm == 1 ? a.km.k_keep % 8 : 0;
  auto cost = [&](int bm, int bn, float far, float tail, TileCost f16, TileCost b16, TileCost f16_seg, TileCost b16_seg) {
    const TileCost c = xm == 2 ? (a.bf16 ? b16_seg : f16_seg) : (a.bf16 ? b16 : f16);
    const long long tiles = (long long)((a.km.n_keep + bn - 1) / bn) * ((a.M + bm - 1) / bm);
    if (bm < 256 && (a.M + bm - 1) / bm > 65535) return 1e30f;   // (a grid row per token tile)
    return launch_cost(tiles, ng, c, a.km.k_span > 8192 ? far : 1.f, tail * (float)odd_columns);
  };
  GemmRoute best = kTile128x256;
  float best_us = cost(128, 256, 1.05f, 4.1f, {1.65f, 0.5f}, {1.85f, 0.4f}, {1.95f, 0.45f}, {2.1f, 0.45f});
  auto take = [&](GemmRoute r, float us) {
    if (us < best_us) best = r, best_us = us;
  };
  // (the pipelined kernel's table is shared by formats and widths; of 4 bits fp16 takes 0.94 of it, bfloat16 0.97)
  if (pipe) take(kPipe, pipe_pick<4>(&a, 1).us * (a.bf16 ? 0.97f : 0.94f));
  if (xm == 1 && prefill_serves(a)) take(kPrefill256, cost(256, 256, 1.05f, 3.9f, {2.75f, 0.8f}, {2.95f, 0.6f}, {}, {}));
  take(kTile64x256, cost(64, 256, 1.05f, 0.85f, {1.03f, 0.22f}, {1.22f, 0.12f}, {1.2f, 0.18f}, {1.4f, 0.13f}));
  take(kTile64x128k2, cost(64, 128, 1.1f, 0.75f, {0.57f, 0.16f}, {0.70f, 0.10f}, {0.78f, 0.14f}, {0.88f, 0.11f}));
  take(kTile32x128k2, cost(32, 128, 1.25f, 0.4f, {0.36f, 0.05f}, {0.47f, 0.05f}, {0.50f, 0.05f}, {0.56f, 0.05f}));
  return best;
}

template <int XVEC, bool BF16>
static hipError_t launch_m(const LinearArgs& a, hipStream_t stream) {
  switch (gemm_route(a, XVEC)) {
    case kSmallM: return smallm_dispatch<XVEC, BF16>(a, stream);
    case kRing: return launch_ring4<BF16>(&a, 1, stream);
    case kPipe: return launch_pipe4<BF16>(&a, 1, stream);
    case kPrefill256:
      if constexpr (XVEC == 1) return launch_prefill_cfg<BF16, 16, 2, 8, 1, 1, 8, 2, 1>(a, stream);
      break;
    // 128 x 256: eight waves side by side over rows, 8 x 2 fragments each, two groups per wave and slab (a block barrier per
    // 256 columns) and two slabs of weight loads in flight (bfloat16: with the longer unpack two do not fit 256 registers)
    case kTile128x256: return launch_cfg<BF16, 8, 2, 8, 1, 2, BF16 ? 1 : 2, XVEC>(a, stream);
    case kTile64x256: return launch_cfg<BF16, 4, 2, 8, 1, 2, 2, XVEC>(a, stream);
    case kTile64x128k2: return launch_cfg<BF16, 4, 2, 4, 2, 2, 1, XVEC>(a, stream);
    case kTile32x128k2: return launch_cfg<BF16, 2, 2, 4, 2, 2, 1, XVEC>(a, stream);
    // (few row tiles: two groups per wave and slab, which halves the number of barriers; many: 32 rows per wave, so that an
    // activation fragment read from LDS serves two weight fragments)
    case kTile16x16k8: return launch_cfg<BF16, 1, 1, 1, 8, 2, 1, XVEC>(a, stream);
    case kTile16x64k4: return launch_cfg<BF16, 1, 2, 2, 4, 1, 2, XVEC>(a, stream);
    case kTile32x16k8: return launch_cfg<BF16, 2, 1, 1, 8, 1, 2, XVEC>(a, stream);
    case kTile32x64k4: return launch_cfg<BF16, 2, 2, 2, 4, 2, 1, XVEC>(a, stream);
    case kTile64x32k4: return launch_cfg<BF16, 4, 1, 2, 4, 1, 2, XVEC>(a, stream);
    case kTile64x64k4: return launch_cfg<BF16, 4, 2, 2, 4, 1, 2, XVEC>(a, stream);
  }
  return hipErrorInvalidValue;
}

// the staging mode of the activations, then the tile shape
static inline int gemm_xm(const LinearArgs& a) {
  // 128-bit x loads: a column prefix (global loads of any size may start on any 2-byte boundary on
  // this target, so odd leading dimensions such as k_keep = 12185 qualify), or column segments
  // whose stride is a multiple of 8 and that keep at least 8 columns each
  if (a.km.cs_stride == 0) return a.km.k_keep >= 8 ? 1 : 0;
  return a.km.cs_stride % 8 == 0 && a.km.cs_keep >= 8 ? 2 : 0;
}

template <bool BF16>
static hipError_t launch_gemm_fmt(const LinearArgs& a, hipStream_t stream) {
  const int xm = gemm_xm(a);
  return xm == 1 ? launch_m<1, BF16>(a, stream) : xm == 2 ? launch_m<2, BF16>(a, stream) : launch_m<0, BF16>(a, stream);
}

// What launch_gemm_fmt (4 bits), the ring and the pipelined kernel (every width) do with a linear of 2 tokens and more, as
// uniql_w4_linear_kernel reports it: the kernel, the tile's tokens and rows and the waves that K is split over (0, 0, 0 for the
// block-staged decode-batch kernel).
static inline void gemm_choice_of(const LinearArgs& a, int out[4]) {
  static const int tiles[][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}, {256, 256, 1}, {128, 256, 1}, {64, 256, 1}, {64, 128, 2}, {32, 128, 2},
                                 {16, 16, 8}, {16, 64, 4}, {32, 16, 8}, {32, 64, 4}, {64, 32, 4}, {64, 64, 4}};
  const int xm = gemm_xm(a);
  const GemmRoute r = a.bits == 4 ? gemm_route(a, xm) : kPipe;
  if (r == kRing || (a.bits != 4 && ring_takes_wide(a))) {
    ring_tile_of(a, out);
    return;
  }
  out[0] = r == kSmallM ? 1 : r == kPipe ? 2 : r == kPrefill256 ? 3 : 4;
  for (int i = 0; i < 3; ++i) out[1 + i] = tiles[r][i];
  if (r != kPipe) return;
  const PipeTile t = a.bits == 4 ? pipe_pick<4>(&a, 1) : a.bits == 8 ? pipe_pick<8>(&a, 1) : a.bits == 6 ? pipe_pick<6>(&a, 1) : pipe_pick<3>(&a, 1);
  out[1] = 16 * t.af;
  out[2] = 16 * t.bf * t.wn;
  out[3] = kPipeConsumers / t.wn;
}

// n (2..4) linears of the same token count and format: those that the decode-batch kernel takes (column prefixes) share a
// launch, and so do those that the pipelined kernel takes with the same split of K and kind of column rule.  Bit i of *left
// stays set for a linear that shares with no other and was not launched.
template <bool BF16>
static hipError_t launch_gemm_batch_fmt(const LinearArgs* a, int n, hipStream_t stream, unsigned* left) {
  // what may share: 1 the decode-batch kernel, 2 and 3 the ring kernel, 4 and up the pipelined one, 0 none
  int kind[kMaxBatch];
  for (int i = 0; i < n; ++i) {
    const int xm = gemm_xm(a[i]);
    const GemmRoute r = gemm_route(a[i], xm);
    kind[i] = r == kSmallM ? (xm == 1 ? 1 : 0) : r == kRing ? 2 + (xm == 2) : r == kPipe ? 4 + pipe_way(a[i]) * 2 + (xm == 2) : 0;
  }
  *left = (1u << n) - 1;
  for (int i = 0; i < n; ++i) {
    if (kind[i] == 0 || !(*left >> i & 1)) continue;
    LinearArgs set[kMaxBatch];
    unsigned taken = 0;
    int m = 0;
    long long outputs = 0;
    for (int j = i; j < n; ++j)
      if (kind[j] == kind[i] && outputs + (long long)a[j].km.n_keep * a[j].M <= kPipeOutputs) {
        set[m++] = a[j], taken |= 1u << j;
        outputs += (long long)a[j].km.n_keep * a[j].M;
      }
    if (m < 2) continue;
    const hipError_t e = kind[i] == 1 ? smallm_batch<BF16>(set, m, stream) : kind[i] <= 3 ? launch_ring4<BF16>(set, m, stream) : launch_pipe4<BF16>(set, m, stream);
    if (e != hipSuccess) return e;
    *left &= ~taken;
  }
  return hipSuccess;
}

}  // namespace uniql
