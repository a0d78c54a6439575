// Host side of the pipelined kernel: what it serves, and how it splits K.
#pragma once
#include "common.h"

namespace uniql {

// Ways to split K over the waves of a block.  The way decides the order of the sums, so it follows from the linear alone,
// never from what it shares a launch with: a linear gives the same bits in a batch and by itself.
//  kPipeGroups : four groups of a slab at a time (KG = 4): up to 32 tokens, and 33..64 on matrices that one round of its tiles of 32
//                tokens takes: 512 row tiles with codes of 3 bits (64-row tiles), 256 with 8 and 6 (32-row ones)
//  kPipeMixed  : two groups, two halves of their steps (KG = KQ = 2): 33..64 tokens, taller matrices (64 or 96 rows x all
//                tokens)
//  kPipeHalves : two halves of a group's steps (KQ = 2): more tokens, 128 x 128 tiles and smaller ones
// 4096 columns at 40 tokens, groups / mixed, with 256, 300, 512, 592 row tiles: 3 bits 10.0 / 15.6, 13.6 / 15.6, 14.7 / 16.4,
// 26.1 / 17.0 us; 8 bits 11.0 / 15.0, 19.3 / 15.3, 20.8 / 16.8, 29.2 / 17.6; 6 bits 13.5 / 17.3, 23.8 / 17.6, 25.1 / 18.5, 35.9 / 19.1;
// 4 bits 9.3 / 13.6, 12.6 / 14.0, 13.5 / 14.6, 24.2 / 15.1.  4 bits change over at 400: such matrices share launches (gate and up, q with k and v), and two of 400..512 row tiles
// are two rounds of the one and one round of the other.
enum PipeWay { kPipeGroups, kPipeMixed, kPipeHalves };

static inline PipeWay pipe_way(const LinearArgs& a) {
  if (a.M > 64) return kPipeHalves;
  const int tall = a.bits == 4 ? 400 : a.bits == 3 ? 513 : 257;   // row tiles
  return a.M > 32 && (a.km.n_keep + 15) / 16 >= tall ? kPipeMixed : kPipeGroups;
}

// Outputs that a launch of the pipelined kernel reaches with its largest tiles (96 tokens x 128 rows and more, 768 threads each: the
// threads of a grid are counted in 32 bits).
constexpr long long kPipeOutputs = 60000000000ll;
constexpr long long kPipeMostThreads = 960;   // of a block, any tile

// At least two tokens, rows of eight groups and more (the window of scales), a column prefix of at least eight columns or
// segments of a power of two up to a group that keep an even number of columns (the last kept pair of x is then a whole
// 32-bit word of its row); 32-bit offsets reach the matrix and a token tile.
static inline bool pipe_serves(const LinearArgs& a) {
  const KeepMap& km = a.km;
  const long long lim = (1ll << 31) - (1 << 17);
  if ((long long)a.km.n_keep * a.M > kPipeOutputs) return false;
  if (a.M < 2 || a.il_heads > 0 || a.K_total < 8 * kGroup) return false;
  if (km.cs_stride == 0 ? km.k_keep < 8 : (km.cs_stride > kGroup || (km.cs_stride & (km.cs_stride - 1)) != 0 || km.cs_keep % 2 != 0)) return false;
  return (long long)a.N_total * (a.K_total / 8) * a.bits < lim && (long long)a.ldx * 2 * 128 + (long long)a.K_total * 2 < lim;
}

// What the ring kernel (ring_kernel.h) serves: 2..32 tokens, rows of eight kept groups and more (one for every wave; the groups that are kept and not the
// stored ones, so that a compact copy of the matrix goes the same way) and up to 320, whose scales and zero points fit the LDS beside the rings; at
// least two rows of fewer than sixteen groups (a window of zero points).
static inline bool ring_serves(const LinearArgs& a) {
  return a.M <= 32 && a.km.k_span > 7 * kGroup && (a.km.k_span > 15 * kGroup || a.km.n_keep > 1) && a.km.k_span <= 320 * kGroup && pipe_serves(a) &&
         ((a.M - 1) * a.ldx + a.km.k_keep) * 2 < (1ll << 31);
}

// Where it is the fastest on 4-bit codes, from 900 sizes timed against the kernels that took them (256..18944 rows, 2048..14336 columns, 2..32 tokens, both
// formats, prefixes and segments; row tiles of 16):
//  - Matrices of fewer than 400 row tiles: prefixes 0.77..0.95 of the time in the mean (0.49..1.05; above 320 row tiles and from 9 tokens
//    on level, and there so that a tall member of a set shares a launch with short ones), segments of up to 16 tokens 0.73..0.88
//    (above 320 row tiles and 8 tokens 1.02).  17..32 tokens of segments 0.82..1.03 up to 256 row tiles, 1.07 above.
//  - 400..600 row tiles: up to 8 tokens 0.77..0.98; 9..32 of prefixes with rows of up to 32 groups 0.88..0.98 above 512, and up to there, one round of the
//    pipelined kernel's 32-row tiles, 0.90..0.99 with up to 20 groups, beyond them 0.97..1.03 at 9..16 tokens and 1.0..1.09 at 17..32.  But two of
//    them in a launch (gate and up) are a full round of the pipelined kernel's 64-row tiles too and four fragments a block here: 9..16 tokens beyond 20 groups
//    1.10..1.20 (8192 x 4096 at 16 tokens 12.1 -> 14.5 us, 7168 x 4096 12.0 -> 14.2), so these are left there, although a set with short ones is then two
//    launches (8192 + 1024 + 1024 x 4096 at 16 tokens 15.7 us, 11.0 in one of this; 16.6 with the short ones in the block-staged kernel).  At 17..32 tokens two are
//    0.94..1.05 and the set 0.65..0.67: they come here.  Longer rows (0.9..1.15) stay with the pipelined kernel, segments of 9..32 tokens (1.02..1.12) with
//    whatever has them.
//  - Taller prefixes with rows of up to 32 groups, by themselves and two of one height in a launch (gate and up).  9..16 tokens: 0.65..0.96
//    and 0.68..0.91 up to 12200 rows and from 16700 to 24000; at 32000 rows 1.01..1.09 (1.05..1.08).  17..32
//    tokens: 0.97..1.08 (0.75..0.82) up to 12200 rows, 0.75..0.82 (0.85..0.99) at 19000 and 24000; 1.04 (1.02..1.04) at 32000.  Between them
//    (769..1024 row tiles: four fragments a block, ring_four) the other kernels fill their rounds: 17..32 tokens 1.10..1.17 (0.86..0.89), 9..16 tokens 0.93..1.12, 1.03 in the
//    mean of 84 sizes (fp16, 4096 columns 1.05..1.12: 14208 rows at 16 tokens 13.2 -> 14.7 us; two in a launch 0.75..0.81): left there, as a linear by itself and in
//    a launch has to take the same kernel.
//  - Up to 8 tokens, prefixes of 601..639 row tiles 0.66..0.99 (160 sizes), and from 640 on, where the block-staged kernel's image of the activations serves
//    rows of up to 32 groups (0.85..1.32 of its time here), longer rows up to 768 row tiles 0.70..0.87, two in a launch 0.64..1.01.  Above that one by itself still is
//    the faster (0.61..1.07), but not two (gate and up; 330 sizes): 769..1024 row tiles 0.80..1.32 (13416 x 11392 at 3 tokens 38.3 -> 50.4 us), 1025..1280 0.70..1.14, and
//    beyond 0.84..1.10 at 2..4 tokens; there from 5 tokens on 0.67..0.98.  Rows of 8..15 groups up to 768 row tiles 0.84..1.04, two 0.84..1.04, beyond 0.75..1.23.
//    Rows of 16..32 groups up to 768 row tiles (576 sizes) where two of these hold: five tokens and more, bfloat16, at most 20 groups: 0.88..1.01, two 0.81..1.02, but
//    others 1.0..1.15 and 0.93..1.08.
//    Where a tall matrix comes here its set with short ones, which are here, is one launch again, which it had stopped being: 10240 + 1024 rows x 5120 columns at
//    8 tokens 22.6 -> 14.7 us (16.4 in one of the block-staged kernel), 12288 + 1024 + 1024 x 12288 43.0 -> 32.9 (41.4), x 2560 12.9 -> 9.9 (10.0).  Others stay two launches:
//    12288 + 1024 + 1024 x 4096 at 2 / 8 tokens 15.8 / 17.5 (14.4 / 15.4 in one of
//    the block-staged kernel, 14.1 in one of this; 14336 + 1024 16.0 / 17.8, 14.6 / 15.6 and 14.4), as by themselves they would lose more here
//    (14336 x 4096 at 8 tokens 11.4 -> 14.1), and 21350 + 2666 + 2666 x 1024 at 5 tokens 11.4 (7.9 in one of the block-staged kernel).  The same at 9..16 tokens with four fragments (14336 + 1024 x 4096 at 16 tokens 19.4, 16.0, 14.9).
//  - Rows of 8..15 groups, prefixes, go by the same lines: 0.49..0.93 up to 375 row tiles (384 sizes), 0.69..1.06 above.  Without them a set of such rows and longer ones
//    was two launches where it had been one: 4096 x 1536 + 4096 x 4096 at 8 / 24 tokens 12.4 / 17.3 -> 8.6 / 9.9 us (9.6 / 16.0 in one of the block-staged
//    kernel), 2048 x 1024 + 1024 x 2048 9.3 / 12.8 -> 4.2 / 5.3 (6.0 / 8.5).  Segments and other widths, which never shared one, stay.
//  - Segments of 17..32 tokens, up to 256 row tiles, beyond 32 groups (460 and 420 sizes): up to 64 groups 0.77..1.05, 0.90 in the mean, bfloat16 and whole blocks as
//    fp16 and partial ones; but 0.94..1.06 on more than 192 row tiles from 25 tokens on, and segments of fewer than 64 columns that keep part of a block
//    (1.04..1.25 on long rows) stay.  65..96 groups up to 192 row tiles 0.77..1.08, 0.90 in the mean; partial blocks in fp16 (0.93..1.03), more row tiles (up to 1.09)
//    and longer rows (up to 1.11) stay.
// (33..64 tokens: a block of 16 rows fetches all of the activations, 29 bytes a clock, which is what takes the time: 0.82 to 1.6, and where
// it was faster by itself the pass of a layer was not.)
constexpr int kRingTallest = 1536;   // row tiles
// One round of the compute units with four fragments a block.  (1025 and 1040 row tiles, five fragments, 9..32 tokens of 4 bits 0.65..0.75 of the time and
// 3 bits 0.63..0.84 where 1024 are 0.98..1.15 and 0.96..1.14.)
static inline bool ring_four(int row_tiles) { return row_tiles > 3 * compute_units() && row_tiles <= 4 * compute_units(); }

static inline bool ring_takes(const LinearArgs& a, bool segments_keep) {   // segments_keep: the block-staged kernel is faster than the pipelined one
  if (a.bits != 4 || !ring_serves(a)) return false;
  const int row_tiles = (a.km.n_keep + 15) / 16, groups = (a.km.k_span + kGroup - 1) / kGroup;
  const bool shorter = groups <= 32;
  if (a.km.cs_stride != 0) {
    if (groups < 16) return false;
    if (a.M <= 8) return row_tiles <= 600;
    if (a.M <= 16) return row_tiles <= 320;
    if (row_tiles > 256) return false;
    if (shorter) return !segments_keep;
    if (a.km.cs_stride < 64 && a.km.cs_keep % 8 != 0) return false;
    if (groups <= 64) return row_tiles <= 192 || a.M <= 24;
    return groups <= 96 && row_tiles <= 192 && !segments_keep;
  }
  if (a.M <= 8) {
    if (row_tiles < 640) return true;
    if (row_tiles <= 3 * compute_units()) return !shorter || groups < 16 || (a.M > 4) + (a.bf16 != 0) + (groups <= 20) >= 2;
    return !shorter && a.M > 4 && row_tiles > 5 * compute_units() && row_tiles <= kRingTallest;
  }
  if (row_tiles < 400) return true;
  if (a.M <= 16 && row_tiles <= 2 * compute_units() && groups > 20) return false;
  return shorter && row_tiles <= kRingTallest && !ring_four(row_tiles);
}

// Codes of 8, 6 and 3 bits: whether the streaming kernel with a token per grid row (w8.hip, wbits.hip) is faster than the pipelined
// one.  It reads and unpacks the weights once per token, but spreads rows and tokens over the whole chip, where the other has a
// block for 32 rows and all tokens: few rows or very few tokens (6 bits, 256 x 12160 at 8 tokens 7.7 against 24.5 us, 2048 x 4096
// at 3 tokens 8.0 against 11.2; 4096 x 4096 at 4 tokens 15.1 against 12.0).  In microseconds, from 1584 timed sizes of 256..131072
// rows, 1024..12185 columns, 2..16 tokens: streaming s0 + s1 kc + (s2 + s3 kc) (rows x tokens / 1000 - 1.5), kc thousands of
// columns (+ s4 with column segments); pipelined p0 + p1 slabs of 512 columns (+ p4), and p2 slabs + p3 more for every further round
// of 256 tiles of 32 rows (3 bits, which have 64-row tiles too: in proportion).  Ties go to the streaming kernel.  The p are
// of an earlier form of the pipelined kernel, which has become faster.  Over 2500 sizes the kernel picked takes 0.2 to 0.9 % longer than
// the faster one in the mean on prefixes and 1.1 to 2.0 % on segments; the worst are matrices of 1000..2000 rows and long segmented
// rows (3 bits, 1024 x 12160, 108 of 128 columns, 11 tokens 35.5 us for 18.9).  Since then the ring kernel has taken what it serves of both from 4096 outputs on
// (ring_takes_wide, below), so this decides up to there, and for rows of up to fifteen groups, matrices of more than 1536 row tiles and the bands that it leaves.
static inline bool wide_streams(const LinearArgs& a) {
  struct Line { float s0, s1, s2, s3, s4, p0, p1, p2, p3, p4; };
  static const Line lines[3][2] = {   // 8, 6, 3 bits; fp16, bfloat16
      {{4.30f, 0.335f, 0.307f, 0.091f, 0.78f, 4.24f, 0.483f, 0.49f, 3.25f, 0.77f}, {4.41f, 0.428f, 0.455f, 0.110f, 0.57f, 4.07f, 0.539f, 0.51f, 3.34f, 0.71f}},
      {{4.00f, 0.417f, 0.157f, 0.114f, 1.81f, 4.65f, 0.936f, 0.91f, 3.20f, 0.66f}, {3.84f, 0.553f, 0.202f, 0.172f, 1.39f, 4.54f, 0.951f, 0.86f, 3.73f, 0.39f}},
      {{4.15f, 0.305f, 0.270f, 0.066f, 0.96f, 3.87f, 0.641f, 0.68f, 1.10f, 0.51f}, {4.40f, 0.409f, 0.436f, 0.119f, 0.41f, 3.88f, 0.686f, 0.78f, 1.07f, 0.48f}}};
  const Line& l = lines[a.bits == 8 ? 0 : a.bits == 6 ? 1 : 2][a.bf16 ? 1 : 0];
  const float seg = a.km.cs_stride != 0 ? 1.f : 0.f, kc = (float)a.km.k_span * 1e-3f, work = (float)a.km.n_keep * (float)a.M * 1e-3f - 1.5f;
  const float slabs = (float)((a.km.k_span + 4 * kGroup - 1) / (4 * kGroup));
  const int tiles = (a.km.n_keep + 31) / 32;
  const float more = a.bits == 3 ? (float)a.km.n_keep / (32.f * 256.f) - 1.f : (float)((tiles + 255) / 256 - 1);
  const float stream = l.s0 + l.s1 * kc + l.s4 * seg + (l.s2 + l.s3 * kc) * (work > 0.f ? work : 0.f);
  const float pipe = l.p0 + l.p1 * slabs + l.p4 * seg + (l.p2 * slabs + l.p3) * (more > 0.f ? more : 0.f);
  return stream < 1.03f * pipe;
}

// Codes of 8, 6 and 3 bits that the ring kernel takes.  From the streaming kernels, which read the weights once per token, where there is more work than
// 4096 outputs (91 sizes that they took, ring / streaming 0.31..0.99, 0.6 in the mean: 2110 x 14336 at 5 tokens, 3 bits, 33.7 -> 11.5 us, 3584 x 18944
// at 2, 6 bits, bfloat16, 43.5 -> 17.1; up to 4096 outputs 0.64..1.39: 1024 x 4096 at 2 tokens, 3 bits, 4.1 for 5.6).  From the pipelined one, whose 32-row tiles leave the chip idle up to 256 row tiles of 16
// and again after every full round of 512, and whose blocks unpack a slab between two barriers.  Over 900 sizes of 512..24000 rows, 2048..18944
// columns, 3..32 tokens, ring / pipelined in the mean: 6 bits 0.64 (up to 16 tokens) and 0.71, 8 bits 0.73..0.85 and 3 bits 0.63..0.84 up to
// 256 row tiles, 0.63..0.82 and 0.66..0.91 above 512 (25..32 tokens on 193..256 row tiles of 33..148 groups 0.68..0.90); us: 18944 x 3584 at 8 tokens, 8 / 6 / 3 bits 21.7 -> 15.4, 29.5 -> 18.0, 21.3 -> 15.1;
// 3584 x 18944 25.0 -> 16.5, 37.7 -> 17.3, 24.1 -> 15.2.  Left where they were:
//  - 257..512 row tiles, one full round of the other's: 8 bits 0.91..1.01, 3 bits 0.97..1.08; 6 bits 0.72..0.90, but 1.07 and 1.09 from 17
//    tokens on with rows of more than 80 groups, whose activations every block fetches.
//  - 3 bits, 769..1024 row tiles (four fragments a block, and the other's second round is full): 0.99..1.13.  More than 1536 row tiles: 0.65..1.09, seven sizes.
static inline bool ring_takes_wide(const LinearArgs& a) {
  if (a.bits == 4 || !ring_serves(a) || a.km.k_span <= 15 * kGroup) return false;
  if (wide_streams(a) && (long long)a.km.n_keep * a.M <= 4096) return false;
  const int row_tiles = (a.km.n_keep + 15) / 16, groups = (a.km.k_span + kGroup - 1) / kGroup;
  if (row_tiles > kRingTallest) return false;
  if (row_tiles > compute_units() && row_tiles <= 2 * compute_units()) return a.bits == 6 && (a.M <= 16 || groups <= 80);
  if (a.bits == 6) return true;
  return a.bits == 8 || !ring_four(row_tiles);
}

}  // namespace uniql
