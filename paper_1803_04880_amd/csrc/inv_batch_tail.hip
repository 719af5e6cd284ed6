// Inverse launch of a batch with partial last rows.
#include "inv_batch_kernel.h"

namespace dwtfrag {

hipError_t launch_inv_batch_tail(const BatchItem *items, const int2 *tiles, int64_t n_tiles,
                                 BatchCounters *ctr, int blocks, hipStream_t s) {
  return launch_inv_batch_t<true>(items, tiles, n_tiles, ctr, blocks, s);
}

}  // namespace dwtfrag
