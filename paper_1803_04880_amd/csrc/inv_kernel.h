// The inverse kernel and its launch (instantiated in two files).
#pragma once

#include "inv.h"

namespace dwtfrag {

// Wavefronts per SIMD that the registers are to allow for: three at 16 columns
// a lane, else four.  (At one level of 8 columns the keystreams' 42.5 KiB of LDS
// a workgroup leave room for three, as the compiler warns.  With three asked for
// it takes as many registers in another order: restore of 16 MiB 28.5 us, with
// four 28.3.)
template <int L, int C1, bool U8OUT, bool TAIL>
__global__ __launch_bounds__(kBlockThreads) __attribute__((amdgpu_waves_per_eu(C1 == 16 ? 3 : 4)))
void inv_kernel(const int16_t *__restrict__ llin, const int16_t *__restrict__ pub,
                void *__restrict__ out, const StageParams P) {
  __shared__ uint32_t s_ks[kWavesPerBlock][inv_ks_words(L, C1)];
  __shared__ uint32_t s_te[1024];
  __shared__ uint32_t s_kw[kKeyWords];
  // the wavefront index is uniform; readfirstlane lets the compiler see that,
  // so all row / level bookkeeping derived from it stays scalar
  const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wave = blockIdx.x * (blockDim.x >> 6) + wib;
  AesLoad aes;
  if (P.use_aes) aes.issue(P.key);
  inv_rect<L, C1, U8OUT, TAIL>(P, wave, llin, pub, out, s_ks[wib], s_te, s_kw, int(threadIdx.x & 63), [&]() {
    aes.finish(s_te, s_kw);
    __syncthreads();
  });
}

template <int L, int C1, bool U8OUT, bool TAIL>
hipError_t launch_inv_t(const int16_t *llin, const int16_t *pub, void *out,
                               const StageParams &P, hipStream_t s) {
  const int per = P.block;
  hipLaunchKernelGGL((inv_kernel<L, C1, U8OUT, TAIL>), dim3((P.n_waves + per - 1) / per), dim3(64 * per), 0,
                     s, llin, pub, out, P);
  return hipGetLastError();
}

}  // namespace dwtfrag
