// Host side of the pipelined kernel: what it serves, and how it splits K.
#pragma once
#include "common.h"

namespace uniql {

// Ways to split K over the waves of a block.  The way decides the order of the sums, so it follows from the linear alone,
// never from what it shares a launch with: a linear gives the same bits in a batch and by itself.
//  kPipeGroups : four groups of a slab at a time (KG = 4): up to 32 tokens, and 33..64 on matrices of fewer than 400 row
//                tiles (32 x 32 tiles give those the most blocks: 656 x 4096 at 48 tokens 8.7 us, 13.6 us in the next way)
//  kPipeMixed  : two groups, two halves of their steps (KG = KQ = 2): 33..64 tokens, taller matrices (64 or 96 rows x all
//                tokens: 9318 x 4096 at 48 tokens 15.0 us, 22.4 us in the way before)
//  kPipeHalves : two halves of a group's steps (KQ = 2): more tokens, 128 x 128 tiles and smaller ones
enum PipeWay { kPipeGroups, kPipeMixed, kPipeHalves };

static inline PipeWay pipe_way(const LinearArgs& a) {
  if (a.M > 64) return kPipeHalves;
  return a.M > 32 && (a.km.n_keep + 15) / 16 >= 400 ? kPipeMixed : kPipeGroups;
}

// At least two tokens, rows of eight groups and more (the window of scales), a column prefix of at least eight columns or
// segments of a power of two up to a group that keep an even number of columns (the last kept pair of x is then a whole
// 32-bit word of its row); 32-bit offsets reach the matrix and a token tile.
static inline bool pipe_serves(const LinearArgs& a) {
  const KeepMap& km = a.km;
  const long long lim = (1ll << 31) - (1 << 17);
  if (a.M < 2 || a.il_heads > 0 || a.K_total < 8 * kGroup) return false;
  if (km.cs_stride == 0 ? km.k_keep < 8 : (km.cs_stride > kGroup || (km.cs_stride & (km.cs_stride - 1)) != 0 || km.cs_keep % 2 != 0)) return false;
  return (long long)a.N_total * (a.K_total / 8) * a.bits < lim && (long long)a.ldx * 2 * 128 + (long long)a.K_total * 2 < lim;
}

}  // namespace uniql
