// Forward launches of single buffers (the streaming code is in fwd.h).
#include "fwd.h"

namespace dwtfrag {

template <int L, int C1, bool U8IN>
__global__ __launch_bounds__(kBlockThreads) __attribute__((amdgpu_waves_per_eu(4))) void fwd_kernel(const void *__restrict__ in,
                                                            int16_t *__restrict__ pub,
                                                            int16_t *__restrict__ llout,
                                                            const StageParams P) {
  __shared__ uint32_t s_ks[kWavesPerBlock][fwd_ks_words(L, C1)];
  __shared__ uint32_t s_te[1024];
  __shared__ uint32_t s_kw[kKeyWords];
  // the wavefront index is uniform; readfirstlane lets the compiler see that,
  // so all row / level bookkeeping derived from it stays scalar
  const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wave = blockIdx.x * (blockDim.x >> 6) + wib;
  AesLoad aes;
  if (P.use_aes) aes.issue(P.key);
  fwd_rect<L, C1, U8IN>(P, wave, in, pub, llout, s_ks[wib], s_te, s_kw, int(threadIdx.x & 63), [&]() {
    aes.finish(s_te, s_kw);
    __syncthreads();
  });
}

template <int L, int C1, bool U8IN>
static hipError_t launch_fwd_t(const void *in, int16_t *pub, int16_t *llout, const StageParams &P,
                               hipStream_t s) {
  const int per = block_waves(P.n_waves);
  hipLaunchKernelGGL((fwd_kernel<L, C1, U8IN>), dim3((P.n_waves + per - 1) / per), dim3(64 * per), 0,
                     s, in, pub, llout, P);
  return hipGetLastError();
}

hipError_t launch_fwd(int L, int C1, bool u8in, const void *in, int16_t *pub, int16_t *llout,
                      const StageParams &P, hipStream_t s) {
#define DWTFRAG_CASE(LL, CC)                                                           \
  if (L == LL && C1 == CC)                                                             \
    return u8in ? launch_fwd_t<LL, CC, true>(in, pub, llout, P, s)                     \
                : launch_fwd_t<LL, CC, false>(in, pub, llout, P, s);
  DWTFRAG_CASE(1, 8) DWTFRAG_CASE(2, 8) DWTFRAG_CASE(3, 8)
  DWTFRAG_CASE(1, 16) DWTFRAG_CASE(2, 16) DWTFRAG_CASE(3, 16) DWTFRAG_CASE(4, 16)
#undef DWTFRAG_CASE
  return hipErrorInvalidValue;
}

}  // namespace dwtfrag
