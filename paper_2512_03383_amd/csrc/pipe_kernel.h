// Linears of more than a few tokens on MFMA for codes of 8, 6, 4 and 3 bits: y[M][n_keep] = x[M][k_keep] * W'^T, with the
// loads in waves of their own.
//
// A block of twelve waves (small tiles: fourteen or fifteen) owns BN = WN * BF * 16 rows and BM = 16 AF tokens.  The columns go by in
// slabs of G groups; a slab is the block's activations and packed codes of those groups.
//  - Two waves (four where the block's registers allow) do nothing but move activations into LDS (128-bit loads that write LDS
//    directly: no registers, no LDS instructions), up to NX - 1 slabs ahead, and one more (two) codes, NW - 1 slabs ahead: loads
//    return in order, and codes come from memory where activations come from the L2.  A mover issues a load every 60 clocks and a
//    CU takes one every 17, so in tiles with little to multiply the moving is what a slab takes: 48 tokens, 35 % of the channels
//    pruned, 148 us a pass of two decoder layers with three movers, 140 with six.  The next slab is there one barrier early (but see XLate).
//  - One wave does the same for scales and zero points, eight groups of a row at a time, through registers.
//  - Eight waves, WN along the rows times KG along the groups of a slab times KQ along the four steps of a group, read codes
//    and activations from LDS, unpack in registers (codes.h) and multiply.  They never wait for memory, and the first
//    fragments of the next slab are read before the barrier that ends the current one.
// The point of the split: in a kernel whose waves load, stage and multiply in turn these phases add up, since all waves
// of a block are in the same phase; here the address unit, the LDS and the matrix pipes work on different slabs at the
// same time.  And a block's share of a packed row is fetched as contiguous runs (17 clocks of the address unit per KB)
// instead of 16 rows per load (65 clocks).
//
// The last round of a grid, where it has at most half as many tiles as there are compute units, goes out as halves: a block takes half the
// tokens of a tile (pipe_half), twice as many compute units have work and it takes 0.8 of the time.  8 bits, 12185 x
// 4096 at 512 tokens, 384 tiles on 256 compute units: 89 -> 83 us, 6 bits 93 -> 80.  The order of the sums is that of any tile.
//
// Codes of 8 bits in 128-token tiles have two slabs on their way, less than the memory's latency: 12185 x 4096 at 512 tokens took 69 us with the
// weights in the 256 MB cache and 83 without.  There the blocks that a die runs side by side on one row tile bring its codes into the L2 a
// window of eight groups ahead (touch), each a quarter of the lines, a dword of each: 83 -> 75 us.  A line costs a compute unit as much as
// its data (29 bytes a clock come in from the L2, whoever asks), so it pays only where four blocks share the work and there is more than
// a round of tiles: 2560 x 2560 at 777 tokens (140 tiles) 21.6 -> 23.2, two or three token tiles 2..9 % slower, 6 and 4 bits level.
//
// LDS layout: activations [token][16 G chunks of 8 columns], chunk c of token t at c ^ bank_key(t); codes [row][units of 16
// bytes], the units of a row permuted likewise where their number is a power of two: the 16 lanes that a 128-bit read serves in
// one clock read 16 different bank groups.  Activations stay in memory order (codes.h gives the weights in that order).
//
// The partial sums of the KG x KQ waves meet in LDS and are added in order; within a wave sums run in order of the columns.  The
// result depends on KG and KQ, not on AF, BF, WN, G, NX or NW.
#pragma once
#include "codes.h"
#include <type_traits>

namespace uniql {

constexpr uint32_t kBufferWord3 = 0x00020000u;
constexpr int kBeyond = (int)0x80000000u;   // as an unsigned offset: past the end of every resource below 2 GiB; reads zeros

constexpr int kPipeConsumers = 8;
constexpr int kPipeTouch = 256;   // bytes of LDS that loads write which only bring lines into the L2
constexpr bool pipe_touches(int bits, int af) { return bits == 8 && af == 8; }
constexpr int kPipeDies = 8, kPipeTokTilesPerPass = 4;

// Up to four linears with the same token count and format; tiles are numbered through the whole batch.
struct PipeBatch {
  LinearArgs p[kMaxBatch];
  int first[kMaxBatch];   // first tile of problem i
  int n, tiles, ntt;      // problems, all tiles, token tiles (the same for every problem)
  int whole;              // tiles that a block takes whole; the rest go out as two halves of the tokens each
  int round;              // tiles of a round: the compute units
};

// HALF: half a tile of a kernel whose blocks have twelve waves
template <int AF, int BF, int WN, int KG, int KQ, int G, int NX, int NW, int BITS, bool SEG, bool HALF = false>
struct PipeShape {
  static_assert(WN * KG * KQ == kPipeConsumers && G == KG && KQ <= 2 && KG * KQ > 1, "eight waves multiply, each one group of a slab, two or all four of its steps");
  static constexpr int BM = 16 * AF, BN = WN * BF * 16, KS = KG * KQ, T = 4 / KQ;   // a wave: T steps of its group
  static constexpr int U = G * BITS;                           // 16-byte units of codes per row and slab
  static constexpr int XBytes = BM * G * 256, WBytes = BN * U * 16;
  static constexpr int XI = XBytes / 1024, WI = WBytes / 1024;   // loads of 64 x 16 bytes
  static constexpr bool Small = !HALF && AF * BF <= 9;
  // (tiles of 16 tokens x 64 rows, 3 and 4 bits, are bound by their codes and lose 1..5 % with more movers, so do 32 x 64 ones of 4 bits on
  // a prefix: 35 sizes of 17..32 tokens, fp16, 1.3 %)
  static constexpr bool MoreMovers = Small && !(BF == 2 && (AF == 1 || (AF == 2 && BITS == 4 && !SEG)));
  static constexpr int XM = MoreMovers ? 4 : 2, WM = MoreMovers && WI % 2 == 0 ? 2 : 1;   // waves that move activations, codes
  // In 32 x 32 tiles of 8-bit codes (a slab is 32 loads of activations and 16 of codes) the codes, which come from memory, must not wait:
  // the two movers of activations that share a SIMD with the movers of codes stand by, and the other two take their loads.
  // 4096 x 12185 at 40 tokens 33.5 -> 26.8 us, x 4096 12.0 -> 10.8 (with the other pair standing by 31.3 and 11.7).  Rows of up to three
  // slabs are mostly the start, which four movers make shorter (4096 x 1024 at 40 tokens 5.4 us, with two 5.7).
  static constexpr bool TwoStandBy = BITS == 8 && AF == 2 && BF == 1;
  static constexpr int MostSlabsOfFour = 3;
  static constexpr int Threads = (kPipeConsumers + XM + WM + 1) * kWave;
  static_assert(WBytes % 1024 == 0 && XI % XM == 0, "whole loads, the same number for each mover");
  static constexpr int XPW = XI / (TwoStandBy ? XM / 2 : XM), WPW = WI / WM;   // (the most that a wave moves of a slab)
  // 8-bit codes in the largest tiles, two slabs in flight: the wave of the scales brings them into the L2 ahead of the movers
  static constexpr bool Touches = pipe_touches(BITS, HALF ? 2 * AF : AF);
  static constexpr int SZ = 2 * BN * 8 * 4;                    // two windows of eight groups
  static constexpr int W0 = NX * XBytes, SZ0 = W0 + NW * WBytes, Lds = SZ0 + SZ + (Touches ? kPipeTouch : 0);
  static_assert((NX - 1) * XPW <= 63 && (NW - 1) * WPW <= 63, "loads in flight are counted in six bits");
  static_assert(NX >= 3 && NW >= 3 && 8 % G == 0 && G <= 4, "a slab in use, one ready, one on its way; a window of scales is two slabs or more");
  static_assert(Lds <= 160 * 1024, "the slabs fit the LDS");
  static_assert(kPipeConsumers * AF * BF * 1024 <= Lds, "so do the partial sums");
};

// What the place of a 16-byte unit in LDS is permuted by, from its token or row.  A 128-bit LDS read serves 16 lanes a clock, and
// these are not 16 consecutive ones: 0-3, 12-15 and 20-27 go together, then 4-11, 16-19 and 28-31 (likewise from lane 32 on; measured
// pair by pair, two lanes of each of eight waves reading one bank at two addresses: 28.2 clocks a read within a set, 24.1 across).  Lane
// l of a fragment reads row l % 16, chunk 4 (l / 16) + t, so rows 0-3 and 12-15 of one chunk share a clock with rows 4-11 of the
// chunk four further on: under r % 16 alone each of these meets one of the former in its bank group (SQ_LDS_BANK_CONFLICT was
// half of the LDS's busy clocks, which were half of all: 8-bit gate at 512 tokens).  With bit 2 of the row added to bit 3 the
// rows that share a clock differ in that bit.
__device__ __forceinline__ int bank_key(int row) { return (row ^ (row << 1 & 8)) & 15; }

__device__ __forceinline__ void pipe_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Half a tile, of AF fragments of tokens (pipe_block.h)
template <int AF, int BF, int WN, int KG, int KQ, int G, int NX, int NW, int BITS, bool BF16, bool SEG>
__device__ __forceinline__ void pipe_half(const LinearArgs& a, int rt, int m0, int share, int mine) {
#ifdef __HIP_DEVICE_COMPILE__   // (the loads into LDS have no form in the host's pass)
  typedef PipeShape<AF, BF, WN, KG, KQ, G, NX, NW, BITS, SEG, true> S;
#include "pipe_block.h"
#endif
}

template <int AF, int BF, int WN, int KG, int KQ, int G, int NX, int NW, int BITS, bool BF16, bool SEG, int HNX>
__global__ __launch_bounds__((PipeShape<AF, BF, WN, KG, KQ, G, NX, NW, BITS, SEG>::Threads), (PipeShape<AF, BF, WN, KG, KQ, G, NX, NW, BITS, SEG>::Small ? 4 : 3)) void w_pipe_kernel(PipeBatch bt) {
#ifdef __HIP_DEVICE_COMPILE__
  typedef PipeShape<AF, BF, WN, KG, KQ, G, NX, NW, BITS, SEG> S;
  constexpr int BM = S::BM, BN = S::BN;
  // Tile of this block.  Consecutive blocks go to the eight dies in turn, each with an L2 of its own: a die takes a
  // contiguous stretch of the tiles, and inside a problem the tiles run row tile by row tile over a few token tiles at
  // a time, so that the blocks a die runs at once share codes and activations through its L2.
  int rt, tt, share, mine, pi = 0, half = 0;
  {
    int b = (int)blockIdx.x, nb = HNX ? bt.whole : bt.tiles, from = 0;
    if (HNX && b >= bt.whole) b -= bt.whole, nb = 2 * (bt.tiles - bt.whole), from = bt.whole, half = 1;
    const int die = b % kPipeDies;
    int L = die * (nb / kPipeDies) + (die < nb % kPipeDies ? die : nb % kPipeDies) + b / kPipeDies;
    if (HNX && half != 0) half += L & 1, L = from + (L >> 1);
#pragma unroll
    for (int i = 1; i < kMaxBatch; ++i) pi += (i < bt.n && L >= bt.first[i]) ? 1 : 0;
    L -= bt.first[pi];
    const int nrt = (bt.p[pi].km.n_keep + BN - 1) / BN, ntt = bt.ntt;
    const int full = ntt / kPipeTokTilesPerPass * kPipeTokTilesPerPass;
    if (L < nrt * full) {
      const int pass = L / (nrt * kPipeTokTilesPerPass), r = L - pass * (nrt * kPipeTokTilesPerPass);
      rt = r / kPipeTokTilesPerPass;
      mine = r - rt * kPipeTokTilesPerPass;
      share = bt.tiles > bt.round ? kPipeTokTilesPerPass : 0;   // (as far as touches go)
      tt = pass * kPipeTokTilesPerPass + mine;
    } else {
      const int w = ntt - full, r = L - nrt * full;
      rt = r / w;
      mine = r - rt * w;
      share = 0;
      tt = full + mine;
    }
  }
  const LinearArgs a = bt.p[pi];
  if constexpr (HNX != 0) {
    if (half != 0) {
      const int m0 = tt * BM + (half - 1) * (BM / 2);
      if (m0 < a.M) pipe_half<AF / 2, BF, WN, KG, KQ, G, HNX, NW, BITS, BF16, SEG>(a, rt, m0, share, mine);
      return;
    }
  }
  const int m0 = tt * BM;
  {
#include "pipe_block.h"
  }
#endif
}

template <int AF, int BF, int WN, int KG, int KQ, int G, int NX, int NW, int BITS, bool SEG, int HNX>
constexpr int pipe_lds() {
  constexpr int whole = PipeShape<AF, BF, WN, KG, KQ, G, NX, NW, BITS, SEG>::Lds;
  if constexpr (HNX != 0) {
    typedef PipeShape<AF / 2, BF, WN, KG, KQ, G, HNX, NW, BITS, SEG, true> Half;
    static_assert(Half::Threads == PipeShape<AF, BF, WN, KG, KQ, G, NX, NW, BITS, SEG>::Threads && AF % 2 == 0, "halves run in the same blocks");
    return Half::Lds > whole ? Half::Lds : whole;
  }
  return whole;
}

// HNX: slabs of activations of half a tile in flight, 0 where there are no halves; whole: tiles that are taken whole (-1: all)
template <int AF, int BF, int WN, int KG, int KQ, int G, int NX, int NW, int BITS, bool BF16, bool SEG, int HNX = 0>
static hipError_t pipe_launch(const LinearArgs* p, int n, hipStream_t stream, int whole = -1) {
  typedef PipeShape<AF, BF, WN, KG, KQ, G, NX, NW, BITS, SEG> S;
  constexpr int lds = pipe_lds<AF, BF, WN, KG, KQ, G, NX, NW, BITS, SEG, HNX>();
  auto kern = w_pipe_kernel<AF, BF, WN, KG, KQ, G, NX, NW, BITS, BF16, SEG, HNX>;
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
  }
  PipeBatch b;
  b.n = n;
  b.ntt = (p[0].M + S::BM - 1) / S::BM;
  int tiles = 0;
  for (int i = 0; i < kMaxBatch; ++i) {
    b.p[i] = p[i < n ? i : 0];
    b.first[i] = tiles;
    if (i < n) tiles += (p[i].km.n_keep + S::BN - 1) / S::BN * b.ntt;
  }
  b.tiles = tiles;
  b.whole = whole < 0 ? tiles : whole;
  b.round = compute_units();
  hipLaunchKernelGGL(kern, dim3(b.whole + 2 * (tiles - b.whole)), dim3(S::Threads), lds, stream, b);
  return hipGetLastError();
}

}  // namespace uniql
