// The forward kernel and its launch (instantiated in two files).
#pragma once

#include "fwd.h"

namespace dwtfrag {

template <int L, int C1, bool U8IN, bool TAIL>
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
  fwd_rect<L, C1, U8IN, TAIL>(P, wave, in, pub, llout, s_ks[wib], s_te, s_kw, int(threadIdx.x & 63), [&]() {
    aes.finish(s_te, s_kw);
    __syncthreads();
  });
}

template <int L, int C1, bool U8IN, bool TAIL>
hipError_t launch_fwd_t(const void *in, int16_t *pub, int16_t *llout, const StageParams &P,
                               hipStream_t s) {
  const int per = P.block;
  hipLaunchKernelGGL((fwd_kernel<L, C1, U8IN, TAIL>), dim3((P.n_waves + per - 1) / per), dim3(64 * per), 0,
                     s, in, pub, llout, P);
  return hipGetLastError();
}

}  // namespace dwtfrag
