// Forward launches of single buffers (the streaming code is in fwd.h).
#include "fwd_kernel.h"

namespace dwtfrag {

hipError_t launch_fwd_tail(int L, int C1, const void *in, int16_t *pub, int16_t *llout,
                           const StageParams &P, hipStream_t s);

hipError_t launch_fwd_few(int L, int C1, bool u8in, const void *in, int16_t *pub, int16_t *llout,
                          const StageParams &P, hipStream_t s);

hipError_t launch_fwd(int L, int C1, bool u8in, const void *in, int16_t *pub, int16_t *llout,
                      const StageParams &P, hipStream_t s) {
  if (few_rows(P, L, C1, true)) return launch_fwd_few(L, C1, u8in, in, pub, llout, P, s);
  // (int16 stages are whole)
  if (P.n_valid < int64_t(P.H) * P.W) return launch_fwd_tail(L, C1, in, pub, llout, P, s);
#define DWTFRAG_CASE(LL, CC)                                                           \
  if (L == LL && C1 == CC)                                                             \
    return u8in ? launch_fwd_t<LL, CC, true, false>(in, pub, llout, P, s)                     \
                : launch_fwd_t<LL, CC, false, false>(in, pub, llout, P, s);
  DWTFRAG_CASE(1, 8) DWTFRAG_CASE(2, 8) DWTFRAG_CASE(3, 8)
  DWTFRAG_CASE(1, 16) DWTFRAG_CASE(2, 16) DWTFRAG_CASE(3, 16) DWTFRAG_CASE(4, 16)
#undef DWTFRAG_CASE
  return hipErrorInvalidValue;
}

}  // namespace dwtfrag
