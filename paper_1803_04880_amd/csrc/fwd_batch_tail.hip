// Forward launch of a batch with partial last rows.
#include "fwd_batch_kernel.h"

namespace dwtfrag {

hipError_t launch_fwd_batch_tail(const BatchItem *items, const int2 *tiles, int64_t n_tiles,
                                 BatchCounters *ctr, int blocks, hipStream_t s) {
  return launch_fwd_batch_t<true>(items, tiles, n_tiles, ctr, blocks, s);
}

}  // namespace dwtfrag
