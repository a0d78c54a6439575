// Which tile of ring_kernel.h a set of linears takes, and its launch.  One translation unit per width and format (ring_w*.hip) instantiates it.
#pragma once
#include "ring_kernel.h"
#include "ring_pick.h"

namespace uniql {

template <int XT, int BITS, bool BF16, bool SEG>
static hipError_t ring_tile(const LinearArgs* p, int n, int bf, hipStream_t s) {
  switch (bf) {
    case 1: return ring_launch<XT, 1, BITS, BF16, SEG>(p, n, s);
    case 2: return ring_launch<XT, 2, BITS, BF16, SEG>(p, n, s);
    case 3: return ring_launch<XT, 3, BITS, BF16, SEG>(p, n, s);
    case 4: return ring_launch<XT, 4, BITS, BF16, SEG>(p, n, s);
    case 5: return ring_launch<XT, 5, BITS, BF16, SEG>(p, n, s);
  }
  if constexpr (!SEG) {
    if (bf == 6) return ring_launch<XT, 6, BITS, BF16, SEG>(p, n, s);
    if constexpr (BITS == 4) {
      if (bf == 7) return ring_launch<XT, 7, BITS, BF16, SEG>(p, n, s);
      if constexpr (XT <= 16) {
        if (bf == 8) return ring_launch<XT, 8, BITS, BF16, SEG>(p, n, s);
      }
    }
  }
  return hipErrorInvalidValue;
}

template <int BITS, bool BF16, bool SEG>
static hipError_t ring_run(const LinearArgs* p, int n, hipStream_t s) {
  const int M = p[0].M, bf = ring_rows(p, n);
  if constexpr (BITS == 4) {
    if (M <= 4) return ring_tile<4, BITS, BF16, SEG>(p, n, bf, s);
  }
  if (M <= 8) return ring_tile<8, BITS, BF16, SEG>(p, n, bf, s);
  if (M <= 16) return ring_tile<16, BITS, BF16, SEG>(p, n, bf, s);
  return ring_tile<32, BITS, BF16, SEG>(p, n, bf, s);
}

// gate (p[0]) and up (p[1]) of 9..16 tokens with h = SiLU(g) * u in one launch (the caller checks that both are served)
template <bool BF16>
static hipError_t ring_glu(const LinearArgs* p, hipStream_t s) {
  return ring_glu_rows(p) == 6 ? ring_launch<16, 6, 4, BF16, false, true>(p, 2, s) : ring_launch<16, 8, 4, BF16, false, true>(p, 2, s);
}

template <int BITS, bool BF16>
static hipError_t ring_linears(const LinearArgs* p, int n, hipStream_t s) {
  return p[0].km.cs_stride != 0 ? ring_run<BITS, BF16, true>(p, n, s) : ring_run<BITS, BF16, false>(p, n, s);
}

}  // namespace uniql
