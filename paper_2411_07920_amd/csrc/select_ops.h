// Digit search of the multi-block radix selections (k_state.hip, k_sort.hip).
#pragma once

#include "swcs_internal.h"

namespace swcs {

// Digit that holds rank k (from the largest) of a histogram that an earlier
// launch counted; false when fewer than k values were.  Called by a whole block;
// *digit, *rest (the rank within the digit) and *held (its count) in every
// thread.  Every block of the next launch searches for itself, 1.5 us from its
// caches, where a last block that waits for all counts, takes a ticket and
// searches added 4 us to every counting launch.
template <int BINS, int THREADS>
__device__ inline bool hist_find(const unsigned* __restrict__ hist, unsigned k, unsigned* s_wave, unsigned* s_pick,
                                 unsigned* digit, unsigned* rest, unsigned* held) {
  constexpr int kPer = BINS / THREADS;
  static_assert(kPer * THREADS == BINS && kPer % 2 == 0, "whole pairs of bins");
  const int t = (int)threadIdx.x, lane = t & 63, wave = t >> 6;
  unsigned h[kPer], sum = 0;
#pragma unroll
  for (int j = 0; j < kPer; ++j) h[j] = hist[BINS - kPer * (t + 1) + j];  // ascending: wide loads
#pragma unroll
  for (int j = 0; j < kPer; ++j) sum += h[j];
  unsigned inc = sum;
  for (int off = 1; off < 64; off <<= 1) {
    const unsigned v = __shfl_up(inc, off);
    if (lane >= off) inc += v;
  }
  if (lane == 63) s_wave[wave] = inc;
  if (t == 0) s_pick[0] = 0xffffffffu;
  __syncthreads();
  unsigned before = inc - sum;
  for (int w = 0; w < wave; ++w) before += s_wave[w];
#pragma unroll
  for (int j = kPer - 1; j >= 0; --j) {
    if (before < k && before + h[j] >= k) {
      s_pick[0] = (unsigned)(BINS - kPer * (t + 1) + j);
      s_pick[1] = k - before;
      s_pick[2] = h[j];
    }
    before += h[j];
  }
  __syncthreads();
  *digit = s_pick[0];
  *rest = s_pick[1];
  *held = s_pick[2];
  return s_pick[0] != 0xffffffffu;
}

}  // namespace swcs
