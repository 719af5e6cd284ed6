// Inverse launches of buffers whose last row is a partial one.
// (At four levels too: 64 MiB of width 8192 less 5 bytes, last segment in the
// general form 105 us, so 60; 17 rows of width 4096 35 against 18.)
#include "inv_kernel.h"

namespace dwtfrag {

hipError_t launch_inv_tail(int L, int C1, const int16_t *llin, const int16_t *pub, void *out,
                           const StageParams &P, hipStream_t s) {
#define DWTFRAG_CASE(LL, CC) \
  if (L == LL && C1 == CC) return launch_inv_t<LL, CC, true, true>(llin, pub, out, P, s);
  DWTFRAG_CASE(1, 8) DWTFRAG_CASE(2, 8) DWTFRAG_CASE(3, 8)
  DWTFRAG_CASE(1, 16) DWTFRAG_CASE(2, 16) DWTFRAG_CASE(3, 16) DWTFRAG_CASE(4, 16)
#undef DWTFRAG_CASE
  return hipErrorInvalidValue;
}

}  // namespace dwtfrag
