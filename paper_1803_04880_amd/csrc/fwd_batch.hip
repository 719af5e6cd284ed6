// Forward launch of a batch.
#include "fwd_batch_kernel.h"

namespace dwtfrag {

hipError_t launch_fwd_batch(const BatchItem *items, const int2 *tiles, int64_t n_tiles,
                            BatchCounters *ctr, int blocks, hipStream_t s) {
  return launch_fwd_batch_t<false>(items, tiles, n_tiles, ctr, blocks, s);
}

// Resident workgroups per CU of the batch forward kernel.
int fwd_batch_blocks_per_cu() {
  int blocks = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, reinterpret_cast<const void *>(&fwd_batch_kernel<false>),
                                                   kBlockThreads, 0) != hipSuccess)
    return 0;
  return blocks;
}

}  // namespace dwtfrag
