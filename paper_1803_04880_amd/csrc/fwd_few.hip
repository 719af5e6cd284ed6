// Forward launches of views of few rows (the code is in fwd_few.h).
#include "batch.h"
#include "fwd_few.h"

namespace dwtfrag {

template <int L, int C1, bool U8IN>
__global__ __launch_bounds__(64) void fwd_few_kernel(const void *__restrict__ in, int16_t *__restrict__ pub,
                                                     int16_t *__restrict__ llout, const StageParams P) {
  __shared__ uint32_t s_ks[kFwdFewKeys<L, C1>];
  __shared__ uint32_t s_te[1024];
  __shared__ uint32_t s_kw[kKeyWords];
  __shared__ uint32_t s_rows[kFwdFewRows<L, C1, U8IN>];
  AesLoad aes;
  if (P.use_aes) aes.issue(P.key);
  fwd_few<L, C1, U8IN>(P, int(blockIdx.x), in, pub, llout, s_ks, s_rows, s_te, s_kw, int(threadIdx.x),
                       [&]() { aes.finish(s_te, s_kw); });
}

template <int L, int C1, bool U8IN>
static hipError_t few(const void *in, int16_t *pub, int16_t *llout, const StageParams &P, hipStream_t s) {
  hipLaunchKernelGGL((fwd_few_kernel<L, C1, U8IN>), dim3(P.n_waves), dim3(64), 0, s, in, pub, llout, P);
  return hipGetLastError();
}

hipError_t launch_fwd_few(int L, int C1, bool u8in, const void *in, int16_t *pub, int16_t *llout,
                          const StageParams &P, hipStream_t s) {
#define DWTFRAG_CASE(LL, CC)                                     \
  if (L == LL && C1 == CC)                                       \
    return u8in ? few<LL, CC, true>(in, pub, llout, P, s) : few<LL, CC, false>(in, pub, llout, P, s);
  DWTFRAG_CASE(1, 8) DWTFRAG_CASE(2, 8) DWTFRAG_CASE(3, 8)
  DWTFRAG_CASE(1, 16) DWTFRAG_CASE(2, 16) DWTFRAG_CASE(3, 16) DWTFRAG_CASE(4, 16)
#undef DWTFRAG_CASE
  return hipErrorInvalidValue;
}

// Batches of such views only: a workgroup of one wavefront per tile.
__global__ __launch_bounds__(64) void fwd_few_batch_kernel(const BatchItem *__restrict__ items,
                                                           const int2 *__restrict__ tiles) {
  __shared__ uint32_t s_ks[kFwdFewKeys<1, kBatchCols>];  // (the most, as are the rows of four levels)
  __shared__ uint32_t s_te[1024];
  __shared__ uint32_t s_kw[kKeyWords];
  __shared__ uint32_t s_rows[kFwdFewRows<4, kBatchCols, true>];
  const int lane = int(threadIdx.x);
  const int2 e = tiles[blockIdx.x];
  const int wave = __builtin_amdgcn_readfirstlane(e.y);
  ConstItem &it = const_items(items)[__builtin_amdgcn_readfirstlane(e.x)];
  const auto tables = [&]() { load_aes_tables(s_te, s_kw, it.fwd.key); };
  const auto go = [&](auto level) {
    fwd_few<decltype(level)::value, kBatchCols, true>(it.fwd, wave, it.in, it.pub, reinterpret_cast<int16_t *>(it.priv),
                                                      s_ks, s_rows, s_te, s_kw, lane, tables);
  };
  switch (it.levels) {
    case 1: go(Level<1>{}); break;
    case 2: go(Level<2>{}); break;
    case 3: go(Level<3>{}); break;
    default: go(Level<4>{}); break;
  }
}

hipError_t launch_fwd_few_batch(const BatchItem *items, const int2 *tiles, int64_t n_tiles, hipStream_t s) {
  hipLaunchKernelGGL(fwd_few_batch_kernel, dim3(unsigned(n_tiles)), dim3(64), 0, s, items, tiles);
  return hipGetLastError();
}

}  // namespace dwtfrag
