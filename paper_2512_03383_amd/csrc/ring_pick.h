// Host side of the ring kernel: the rows of a block.
#pragma once
#include "common.h"

namespace uniql {

// tokens of a slot of activations (four: only where 4-bit codes make them a part of the traffic that counts)
static inline int ring_tokens(int M, int bits) { return M <= 4 && bits == 4 ? 4 : M <= 8 ? 8 : M <= 16 ? 16 : 32; }

// LDS of a block: what ring_kernel.h's RingShape says for the codes, the activations, the scales and zero points of bf fragments of 16
// rows, or the partial sums
constexpr int kRingLds = 160 * 1024;

// Fragments of 16 rows per block: the fewest rounds of the chip's compute units (a block fills one), then the fewest rows: a round costs
// its fragments and one more (14208 x 3584 at 8 tokens, 888 row tiles, 1 .. 5 fragments 19.6, 16.0, 18.5, 13.3, 13.7 us; 14336 x 4096 at 32
// tokens 28.4, 19.5, 23.2, 15.8, 17.4; two of 14336 x 4096 at 16 tokens, 3 .. 8 fragments 30.1, 27.4, 31.2, 30.0, 21.4, 22.3).  Beyond five
// a launch of column segments has not been found faster; eight of 32 tokens do not fit the LDS; wide codes do
// not come in launches of several matrices, and one of up to 1536 row tiles never wants more than six.  The order of the sums does not depend on it.
static inline int ring_rows(const LinearArgs* p, int n) {
  const int cus = compute_units(), most = p[0].km.cs_stride != 0 ? 5 : p[0].bits != 4 ? 6 : p[0].M <= 16 ? 8 : 7;
  int groups = 0;
  for (int i = 0; i < n; ++i) groups = (p[i].km.k_span + kGroup - 1) / kGroup > groups ? (p[i].km.k_span + kGroup - 1) / kGroup : groups;
  int best = 1;
  float best_cost = 1e30f;
  for (int bf = 1; bf <= most; ++bf) {
    // (18 KB a wave for its ring; long rows do not leave room for the scales of many rows)
    if (bf > 1 && 8 * 18 * 1024 + ((groups + 7) / 8 + (groups + 15) / 16) * bf * 256 + 256 > kRingLds) break;
    long long tiles = 0;
    for (int i = 0; i < n; ++i) tiles += (p[i].km.n_keep + 16 * bf - 1) / (16 * bf);
    const float cost = (float)((tiles + cus - 1) / cus) * ((float)bf + 1.f);
    if (cost < best_cost) best = bf, best_cost = cost;
  }
  return best;
}

// the same for a gated pair: three or four fragments of each matrix (the pairs that are served have 640 .. 1536 row tiles: fewer never are the best)
static inline int ring_glu_rows(const LinearArgs* p) {
  const int cus = compute_units(), row_tiles = (p[0].km.n_keep + 15) / 16;
  auto rounds = [&](int rows) { return ((row_tiles + rows - 1) / rows + cus - 1) / cus; };
  return rounds(3) * 7 <= rounds(4) * 9 ? 6 : 8;
}

// as uniql_w4_linear_kernel reports it, for every width and column rule: a decode-batch kernel, tokens and rows of a tile, K over eight waves
static inline void ring_tile_of(const LinearArgs& a, int out[4]) {
  out[0] = 1, out[1] = ring_tokens(a.M, a.bits), out[2] = 16 * ring_rows(&a, 1), out[3] = 8;
}

}  // namespace uniql
