// Forward batch kernel (instantiated in two files; the streaming code is in fwd.h).
#pragma once

#include "batch.h"
#include "fwd.h"

namespace dwtfrag {

// Batch form: one persistent launch drains the batch's tile queue; each tile
// is one wavefront rectangle of one item (the item's own plan, buffers and
// keys), run by the streaming code of the item's depth.
constexpr int cmax(int a, int b) { return a > b ? a : b; }
constexpr int kFwdBatchKs = cmax(cmax(fwd_ks_words(1, kBatchCols), fwd_ks_words(2, kBatchCols)),
                                 cmax(fwd_ks_words(3, kBatchCols), fwd_ks_words(4, kBatchCols)));

template <int L, bool TAIL>
__device__ __forceinline__ void fwd_batch_tile(ConstItem &it, int wave, uint32_t *ks,
                                               const uint32_t *te, const uint32_t *kw, int lane) {
  fwd_rect<L, kBatchCols, true, TAIL>(it.fwd, wave, it.in, it.pub, reinterpret_cast<int16_t *>(it.priv), ks,
                                te, kw, lane, [] {});
}

template <bool TAIL>
__global__ __launch_bounds__(kBlockThreads) void fwd_batch_kernel(const BatchItem *__restrict__ items,
                                                                  const int2 *__restrict__ tiles,
                                                                  int64_t n_tiles,
                                                                  BatchCounters *__restrict__ ctr) {
  __shared__ uint32_t s_ks[kWavesPerBlock][kFwdBatchKs];
  __shared__ uint32_t s_te[1024];
  __shared__ uint32_t s_kw[kWavesPerBlock][kKeyWords];
  load_aes_te(s_te);
  __syncthreads();
  const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  for (;;) {
    unsigned int t = 0;
    if (lane == 0) t = atomicAdd(&ctr->head, 1u);
    t = __builtin_amdgcn_readfirstlane(t);
    if (int64_t(t) >= n_tiles) break;
    const int2 e = tiles[t];
    const int wave = __builtin_amdgcn_readfirstlane(e.y);
    ConstItem &it = const_items(items)[__builtin_amdgcn_readfirstlane(e.x)];
    if (lane < kKeyWords) s_kw[wib][lane] = key_word(it.fwd.key, lane);  // this item's keys
    wave_lds_sync();
    switch (it.levels) {
      case 1: fwd_batch_tile<1, TAIL>(it, wave, s_ks[wib], s_te, s_kw[wib], lane); break;
      case 2: fwd_batch_tile<2, TAIL>(it, wave, s_ks[wib], s_te, s_kw[wib], lane); break;
      case 3: fwd_batch_tile<3, TAIL>(it, wave, s_ks[wib], s_te, s_kw[wib], lane); break;
      default: fwd_batch_tile<4, TAIL>(it, wave, s_ks[wib], s_te, s_kw[wib], lane); break;
    }
    wave_lds_sync();
  }
  batch_finish(ctr);
}

template <bool TAIL>
hipError_t launch_fwd_batch_t(const BatchItem *items, const int2 *tiles, int64_t n_tiles, BatchCounters *ctr,
                              int blocks, hipStream_t s) {
  hipLaunchKernelGGL(fwd_batch_kernel<TAIL>, dim3(blocks), dim3(kBlockThreads), 0, s, items, tiles,
                     n_tiles, ctr);
  return hipGetLastError();
}

}  // namespace dwtfrag
