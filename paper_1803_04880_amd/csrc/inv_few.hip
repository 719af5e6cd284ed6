// Inverse launches of views of few rows (the code is in inv_few.h).
#include "batch.h"
#include "inv_few.h"

namespace dwtfrag {

template <int L, int C1, bool U8OUT, bool GEN>
__global__ __launch_bounds__(64) void inv_few_kernel(const int16_t *__restrict__ llin, const int16_t *__restrict__ pub,
                                                     void *__restrict__ out, const StageParams P) {
  __shared__ uint32_t s_ks[kInvFewKeys<L, C1>];
  __shared__ uint32_t s_te[1024];
  __shared__ uint32_t s_kw[kKeyWords];
  extern __shared__ uint32_t s_rows[];  // by the view's rows
  AesLoad aes;
  if (P.use_aes) aes.issue(P.key);
  inv_few<L, C1, U8OUT, GEN>(P, int(blockIdx.x), llin, pub, out, s_ks, s_rows, s_te, s_kw, int(threadIdx.x),
                             [&]() { aes.finish(s_te, s_kw); });
}

template <int L, int C1, bool U8OUT>
static hipError_t few(const int16_t *llin, const int16_t *pub, void *out, const StageParams &P, hipStream_t s) {
  const unsigned lds = inv_few_lds(P, L, C1);
  if (P.W % C1)
    hipLaunchKernelGGL((inv_few_kernel<L, C1, U8OUT, true>), dim3(P.n_waves), dim3(64), lds, s, llin, pub, out, P);
  else
    hipLaunchKernelGGL((inv_few_kernel<L, C1, U8OUT, false>), dim3(P.n_waves), dim3(64), lds, s, llin, pub, out, P);
  return hipGetLastError();
}

hipError_t launch_inv_few(int L, int C1, bool u8out, const int16_t *llin, const int16_t *pub, void *out,
                          const StageParams &P, hipStream_t s) {
#define DWTFRAG_CASE(LL, CC)                                       \
  if (L == LL && C1 == CC)                                         \
    return u8out ? few<LL, CC, true>(llin, pub, out, P, s) : few<LL, CC, false>(llin, pub, out, P, s);
  DWTFRAG_CASE(1, 8) DWTFRAG_CASE(2, 8) DWTFRAG_CASE(3, 8)
  DWTFRAG_CASE(1, 16) DWTFRAG_CASE(2, 16) DWTFRAG_CASE(3, 16) DWTFRAG_CASE(4, 16)
#undef DWTFRAG_CASE
  return hipErrorInvalidValue;
}

// Batches of such views only: a workgroup of one wavefront per tile.  (One
// form, the general one: a second of every depth would double the code.)
__global__ __launch_bounds__(64) void inv_few_batch_kernel(const BatchItem *__restrict__ items,
                                                           const int2 *__restrict__ tiles) {
  __shared__ uint32_t s_ks[kInvFewKeys<1, kBatchCols>];  // (the most)
  __shared__ uint32_t s_te[1024];
  __shared__ uint32_t s_kw[kKeyWords];
  extern __shared__ uint32_t s_rows[];  // by the batch's tallest
  const int lane = int(threadIdx.x);
  const int2 e = tiles[blockIdx.x];
  const int wave = __builtin_amdgcn_readfirstlane(e.y);
  ConstItem &it = const_items(items)[__builtin_amdgcn_readfirstlane(e.x)];
  const auto tables = [&]() { load_aes_tables(s_te, s_kw, it.inv.key); };
  const auto go = [&](auto level) {
    inv_few<decltype(level)::value, kBatchCols, true, true>(it.inv, wave, reinterpret_cast<const int16_t *>(it.priv),
                                                            it.pub, it.out, s_ks, s_rows, s_te, s_kw, lane, tables);
  };
  switch (it.levels) {
    case 1: go(Level<1>{}); break;
    case 2: go(Level<2>{}); break;
    case 3: go(Level<3>{}); break;
    default: go(Level<4>{}); break;
  }
}

hipError_t launch_inv_few_batch(const BatchItem *items, const int2 *tiles, int64_t n_tiles, unsigned lds,
                                hipStream_t s) {
  hipLaunchKernelGGL(inv_few_batch_kernel, dim3(unsigned(n_tiles)), dim3(64), lds, s, items, tiles);
  return hipGetLastError();
}

}  // namespace dwtfrag
