// Inverse launches of single buffers (the streaming code is in inv.h).
#include "inv_kernel.h"

namespace dwtfrag {

hipError_t launch_inv_tail(int L, int C1, const int16_t *llin, const int16_t *pub, void *out,
                           const StageParams &P, hipStream_t s);

hipError_t launch_inv_few(int L, int C1, bool u8out, const int16_t *llin, const int16_t *pub, void *out,
                          const StageParams &P, hipStream_t s);

hipError_t launch_inv(int L, int C1, bool u8out, const int16_t *llin, const int16_t *pub,
                      void *out, const StageParams &P, hipStream_t s) {
  if (few_rows(P, L, C1, false)) return launch_inv_few(L, C1, u8out, llin, pub, out, P, s);
  // (int16 stages are whole)
  if (P.n_valid < int64_t(P.H) * P.W) return launch_inv_tail(L, C1, llin, pub, out, P, s);
#define DWTFRAG_CASE(LL, CC)                                                   \
  if (L == LL && C1 == CC)                                                     \
    return u8out ? launch_inv_t<LL, CC, true, false>(llin, pub, out, P, s)            \
                 : launch_inv_t<LL, CC, false, false>(llin, pub, out, P, s);
  DWTFRAG_CASE(1, 8) DWTFRAG_CASE(2, 8) DWTFRAG_CASE(3, 8)
  DWTFRAG_CASE(1, 16) DWTFRAG_CASE(2, 16) DWTFRAG_CASE(3, 16) DWTFRAG_CASE(4, 16)
#undef DWTFRAG_CASE
  return hipErrorInvalidValue;
}

}  // namespace dwtfrag
