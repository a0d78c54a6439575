// Which tile of pipe_kernel.h a linear takes, and its launch.  One translation unit per code width and format
// (pipe_w*.hip) instantiates it.
#pragma once
#include "pipe_kernel.h"
#include "pipe_serves.h"

namespace uniql {

// What a launch costs, in microseconds: a group of 128 columns (or a slab of them) costs one tile `us` on an idle chip and
// `slope` more with every compute unit busy (clock and L2), a round of tiles 4 besides and `round` more, the launch 3.  Rows of
// more than 8192 columns miss the L2 more often.  It ranks tiles; as a time it is rough.  The costs of a prefix, and all of up to 64 tokens, are of an
// earlier form of the pipelined kernel and lie above its times now, those of segments at more tokens are of the present one: with every
// tile timed at 1591 sizes (1024..28672 rows, 1024..14208 columns, 72..2048 tokens, all widths and formats, prefixes and 108 of 128
// columns) a tile took 0.74..1.12 of its cost (5th to 95th percentile; median 0.84 for a prefix in 4 and 8 bits, 0.94 for segments).  The
// tile picked takes 0.1 % longer than the fastest one in the mean and 6 % at worst; with 8 bits 0.2 %, and 13 % (6000 x 14208 at 1000
// tokens 230 us in 64 x 128 tiles, 203 in 128 x 128) to 17 % at worst (12185 x 14208, segments, 512 tokens: 296 in 128 x 128, 253 in 64 x 128).
// Up to 64 tokens (809 sizes) 0.0 % in the mean, 5 % at worst.
struct TileCost {
  float us, slope;
};
static inline float launch_cost(long long tiles, float steps, TileCost c, float far, float round = 0.f) {
  const int cus = compute_units();
  const float rounds = (float)((tiles + cus - 1) / cus);
  return 3.f + rounds * (4.f + round + steps * (c.us + c.slope * (float)tiles / (rounds * (float)cus)) * far);
}

struct PipeTile {
  int af, bf, wn, g;
  TileCost prefix, seg;   // per slab of g groups
  float us;               // of the launch
  int whole;              // tiles that are taken whole, -1: all (the others as two halves of the tokens)
};

// Tiles of this many fragments of 16 tokens have halves (of 64 and 48 tokens; their blocks have the same waves and the same LDS).  8-bit
// codes: not those of 96 tokens, which the shared costs rate too well against 128 (12185 x 4096, 108 of 128 columns, 200 tokens
// 41.5 us in 128-token tiles, 44.6 in 96 with halves).
constexpr bool pipe_halves(int bits, int af) { return af == 8 || (af == 6 && bits != 8); }

template <int BITS>
static inline PipeTile pipe_pick(const LinearArgs* p, int n) {
  // groups: 32- and 64-row tiles; mixed: 64- and 96-row tiles (96 rows x 64 tokens do not fit with 8-bit codes);
  // halves: rows x tokens from 128 x 128 down to 64 x 64 (8-bit codes: no 112, its buffers)
  // (128 x 128 takes all of a wave's 168 registers: with 8 and 6 bits a word (fp16) or up to five (bfloat16) goes to scratch around
  // the loop, and 2 to 17 words in the loop of the bfloat16 unpack's wide form)
  static const PipeTile groups[] = {{1, 1, 2, 4, {0.50f, 0.05f}, {0.55f, 0.05f}, 0.f, -1}, {1, 2, 2, 4, {0.90f, 0.05f}, {0.95f, 0.05f}, 0.f, -1},
                                    {2, 1, 2, 4, {0.55f, 0.05f}, {0.65f, 0.05f}, 0.f, -1}, {2, 2, 2, 4, {1.0f, 0.05f}, {1.05f, 0.05f}, 0.f, -1}};
  static const PipeTile mixed[] = {{3, 2, 2, 2, {0.62f, 0.07f}, {0.70f, 0.05f}, 0.f, -1}, {3, 3, 2, 2, {0.80f, 0.07f}, {0.90f, 0.05f}, 0.f, -1},
                                   {4, 2, 2, 2, {0.73f, 0.07f}, {0.85f, 0.05f}, 0.f, -1}, {4, 3, 2, 2, {0.93f, 0.07f}, {1.05f, 0.05f}, 0.f, -1}};
  static const PipeTile halves[] = {{8, 2, 4, 1, {1.0f, 0.15f}, {0.82f, 0.22f}, 0.f, -1}, {7, 2, 4, 1, {0.93f, 0.12f}, {0.76f, 0.12f}, 0.f, -1},
                                    {6, 2, 4, 1, {0.85f, 0.07f}, {0.71f, 0.09f}, 0.f, -1}, {4, 2, 4, 1, {0.56f, 0.15f}, {0.58f, 0.07f}, 0.f, -1},
                                    {4, 1, 4, 1, {0.33f, 0.09f}, {0.33f, 0.04f}, 0.f, -1}};
  const PipeWay way = pipe_way(p[0]);
  const bool seg = p[0].km.cs_stride != 0;
  const PipeTile* set = way == kPipeGroups ? groups : way == kPipeMixed ? mixed : halves;
  const int count = way == kPipeHalves ? 5 : 4, M = p[0].M;
  int span = 0;
  for (int i = 0; i < n; ++i) span = p[i].km.k_span > span ? p[i].km.k_span : span;
  const int ngroups = (span + kGroup - 1) / kGroup;
  PipeTile best = {};
  for (int c = 0; c < count; ++c) {
    PipeTile t = set[c];
    if (way == kPipeGroups && t.af != (M <= 16 ? 1 : 2)) continue;
    if (way == kPipeMixed && t.af != (M <= 48 ? 3 : 4)) continue;
    if (BITS > 4 && way != kPipeGroups && ((t.af == 4 && t.bf == 3) || t.af == 7)) continue;
    if (BITS > 4 && way == kPipeGroups && t.bf == 2) continue;
    long long tiles = 0;
    for (int i = 0; i < n; ++i) tiles += (p[i].km.n_keep + t.wn * t.bf * 16 - 1) / (t.wn * t.bf * 16);
    tiles *= (M + 16 * t.af - 1) / (16 * t.af);
    // (threads of a grid are counted in 32 bits; pipe_serves leaves the largest tiles below that)
    t.us = tiles * kPipeMostThreads >= (1ll << 32) ? 1e30f : launch_cost(tiles, (float)((ngroups + t.g - 1) / t.g), seg ? t.seg : t.prefix, span > 8192 ? 1.18f : 1.f);
    // A last round of at most half as many tiles as there are compute units goes out as halves of the tokens, two blocks a tile.  Such a
    // round takes 0.78 (128 tokens) or 0.82 (96) of a whole one, with 500 sizes timed both ways (1.1 .. 8 rounds, all widths): the launch
    // 0.85 to 0.997 of the time.  The costs here are a little above, so that another tile is not left for too small a gain.  Prefixes of 4 and 3 bits have 112-token
    // tiles, whose two rounds were rated level with one of 128 tokens and its halves but are the faster on long rows (54 such sizes 0.91 to 1.04 of their time; 11642 x
    // 5376 at 491 tokens 85.9 us, 94.8 in halves): one more, and halves are left to where they gain (11843 x 3200 twice at 255 tokens 73.3 -> 61.5).
    if (way == kPipeHalves && pipe_halves(BITS, t.af) && tiles < (1 << 20)) {
      const int cus = compute_units(), rest = (int)(tiles % cus);
      if (tiles > cus && rest > 0 && 2 * rest <= cus) {
        const TileCost& c = seg ? t.seg : t.prefix;
        const float steps = (float)((ngroups + t.g - 1) / t.g), far = span > 8192 ? 1.18f : 1.f;
        const float us = launch_cost(tiles - rest, steps, c, far) + (t.af != 8 ? 0.88f : BITS <= 4 && !seg ? 0.87f : 0.8f) * (4.f + steps * (c.us + c.slope) * far);
        if (us < t.us) t.us = us, t.whole = (int)tiles - rest;
      }
    }
    if (best.af == 0 || t.us < best.us) best = t;
  }
  return best;
}

// slabs of codes in flight where the activations leave room
constexpr int pipe_nw(int lds, int sz, int wbytes, int most) {
  int n = (160 * 1024 - lds - sz) / wbytes;
  n = n < most ? n : most;
  const int counted = 63 / (wbytes / 1024) + 1;   // (n - 1 slabs of loads in flight are counted in six bits)
  return n < counted ? n : counted;
}
template <int AF, int BF, int WN, int KG, int KQ, int G, int NX, int BITS, bool BF16, bool SEG>
static hipError_t pipe_tile(const LinearArgs* p, int n, hipStream_t s, int whole = -1) {
  constexpr int BN = WN * BF * 16;
  constexpr int NW = pipe_nw(NX * 16 * AF * G * 256, BN * 64 + (pipe_touches(BITS, AF) ? kPipeTouch : 0), BN * G * BITS * 16, 8);
  static_assert(PipeShape<AF, BF, WN, KG, KQ, G, NX, NW, BITS, SEG>::Threads <= kPipeMostThreads, "pipe_pick counts the threads of a grid with the largest block");
  // (a slab of half the tokens is half as long: the same LDS)
  return pipe_launch<AF, BF, WN, KG, KQ, G, NX, NW, BITS, BF16, SEG, pipe_halves(BITS, AF) ? 2 * NX : 0>(p, n, s, whole);
}

template <int BITS, bool BF16, bool SEG>
static hipError_t pipe_run(const LinearArgs* p, int n, hipStream_t s) {
  const PipeTile t = pipe_pick<BITS>(p, n);
  switch (pipe_way(p[0])) {
    case kPipeGroups:
      if constexpr (BITS <= 4) {
        if (t.bf == 2) return t.af == 1 ? pipe_tile<1, 2, 2, 4, 1, 4, 3, BITS, BF16, SEG>(p, n, s) : pipe_tile<2, 2, 2, 4, 1, 4, 3, BITS, BF16, SEG>(p, n, s);
      }
      return t.af == 1 ? pipe_tile<1, 1, 2, 4, 1, 4, 4, BITS, BF16, SEG>(p, n, s) : pipe_tile<2, 1, 2, 4, 1, 4, 3, BITS, BF16, SEG>(p, n, s);
    case kPipeMixed:
      if (t.af == 3) return t.bf == 2 ? pipe_tile<3, 2, 2, 2, 2, 2, BITS <= 4 ? 4 : 3, BITS, BF16, SEG>(p, n, s) : pipe_tile<3, 3, 2, 2, 2, 2, 3, BITS, BF16, SEG>(p, n, s);
      if constexpr (BITS <= 4) {
        if (t.bf == 3) return pipe_tile<4, 3, 2, 2, 2, 2, 3, BITS, BF16, SEG>(p, n, s);
      }
      return pipe_tile<4, 2, 2, 2, 2, 2, 3, BITS, BF16, SEG>(p, n, s);
    default:
      if (t.af == 8) return pipe_tile<8, 2, 4, 1, 2, 1, 3, BITS, BF16, SEG>(p, n, s, t.whole);
      if constexpr (BITS <= 4) {
        if (t.af == 7) return pipe_tile<7, 2, 4, 1, 2, 1, 4, BITS, BF16, SEG>(p, n, s);
      }
      if (t.af == 6) return pipe_tile<6, 2, 4, 1, 2, 1, BITS <= 4 ? 4 : 3, BITS, BF16, SEG>(p, n, s, t.whole);
      return t.bf == 2 ? pipe_tile<4, 2, 4, 1, 2, 1, BITS == 8 ? 4 : 6, BITS, BF16, SEG>(p, n, s) : pipe_tile<4, 1, 4, 1, 2, 1, 6, BITS, BF16, SEG>(p, n, s);
  }
}

// n linears (the same token count, format, width, way and kind of column rule; the caller checks) in one launch
template <int BITS, bool BF16>
static hipError_t pipe_linears(const LinearArgs* p, int n, hipStream_t s) {
  return p[0].km.cs_stride != 0 ? pipe_run<BITS, BF16, true>(p, n, s) : pipe_run<BITS, BF16, false>(p, n, s);
}

}  // namespace uniql
