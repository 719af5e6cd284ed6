// Per-row inverse lifting in 32-bit arithmetic, for the stream that redoes
// rectangles outside the packed range.
//
// Lane layout: at level l a lane holds C = C1 >> (l-1) consecutive samples of
// the level-(l-1) LL row, indices j0 .. j0+C-1 with j0 even.  Even positions
// are lows, odd positions highs (Ch. 5 eqs. (5.1)-(5.2)).  The neighbour
// beyond the lane's last sample comes from the next lane, the one before its
// first sample from the previous lane (one DPP move each).
#pragma once

#include "common.h"

namespace dwtfrag {

// Undo the update on even positions, eq. (5.2) additive, then the predict on
// odd ones, eq. (5.1).  EDGE: the wavefront covers index 0 or N-1, where
// whole-sample mirroring replaces the missing neighbour by the one on the
// other side.
template <int C, bool EDGE>
__device__ __forceinline__ void hinv(int (&v)[C], int j0, int N) {
  const int left_d = from_prev_lane(v[C - 1]);
#pragma unroll
  for (int t = 0; t < C; t += 2) {
    int l = (t > 0) ? v[t - 1] : left_d;
    int r = v[t + 1];
    if (EDGE) {
      if (j0 + t == 0) l = r;
      if (j0 + t == N - 1) r = l;
    }
    v[t] -= (l + r + 2) >> 2;
  }
  const int right0 = from_next_lane(v[0]);
#pragma unroll
  for (int t = 1; t < C; t += 2) {
    int r = (t + 1 < C) ? v[t + 1] : right0;
    if (EDGE && j0 + t == N - 1) r = v[t - 1];
    v[t] += (v[t - 1] + r) >> 1;
  }
}

template <int C>
__device__ __forceinline__ void hinv_any(int (&v)[C], int j0, int N, bool edge) {
  if (N == 1) return;
  if (edge) hinv<C, true>(v, j0, N);
  else hinv<C, false>(v, j0, N);
}

}  // namespace dwtfrag
