// Device-side tables of a batch of independent buffers (protect / restore of
// many chunks in one go: the thesis cuts data into many equal chunks, Ch. 5
// section 5.2.1, and its GPU runs take many chunks as input).
//
// Each buffer ("item") is one fused stage (levels <= 4) planned with 16
// columns per lane, the layout every depth up to four levels can use, so one
// kernel per direction serves all items: its tiles (item, wavefront index
// within the item) form a single queue, longest first, that one persistent
// launch drains with an atomic head counter, dispatching each tile on its
// item's depth.  The last workgroup to finish resets the counters, so a
// batch direction is exactly one kernel launch.
#pragma once

#include "common.h"

namespace dwtfrag {

// Columns per lane of every batch tile.
constexpr int kBatchCols = 16;

// A depth, to pick a kernel's code by.
template <int L> struct Level { static constexpr int value = L; };

struct BatchItem {
  StageParams fwd;     // forward plan (halo shape of the forward kernel)
  StageParams inv;     // inverse plan
  const uint8_t *in;   // protect input (device)
  uint8_t *priv;       // private fragment (device)
  int16_t *pub;        // public fragment (device)
  uint8_t *out;        // restore output (device)
  uint64_t priv_bytes; // 2 * h_L * w_L
  int32_t levels;      // 1..4
  int32_t pad;
};

// The item table as the kernels read it: by scalar loads (it is written
// before the launch).
using ConstItem = const __attribute__((address_space(4))) BatchItem;
__device__ __forceinline__ ConstItem *const_items(const BatchItem *items) { return (ConstItem *)items; }

// Queue counters of one direction: [0] next tile, [1] finished workgroups.
struct BatchCounters {
  unsigned int head, done;
};

// The tiles of one item in a direction's queue: they follow one another from
// tile `first` of the table on.  The tables of both directions are one, in
// queue order; a plan's host side makes only these runs, and the tile list is
// written on the device (batch_tiles_kernel).
struct BatchRun {
  int64_t first;
  int32_t item, pad;
};

// Tile t of the n runs: (item, wavefront index within the item).
__host__ __device__ inline int2 batch_tile(const BatchRun *runs, int64_t n, int64_t t) {
  int64_t lo = 0, hi = n;  // the last run that begins at or before t
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) / 2;
    if (runs[mid].first <= t) lo = mid;
    else hi = mid;
  }
  return make_int2(runs[lo].item, int(t - runs[lo].first));
}

// Called by every workgroup once its wavefronts have left the tile loop: the
// last one resets both counters for the next launch (no other workgroup pops
// a tile any more at that point).
__device__ __forceinline__ void batch_finish(BatchCounters *c) {
  __syncthreads();
  if (threadIdx.x == 0) {
    __threadfence();
    const unsigned int d = atomicAdd(&c->done, 1u);
    if (d == gridDim.x - 1) {
      atomicExch(&c->head, 0u);
      atomicExch(&c->done, 0u);
    }
  }
}

}  // namespace dwtfrag
