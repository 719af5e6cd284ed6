// Forward launches of buffers whose last row is a partial one.
// (At four levels the checks spill 160 bytes a lane where the kernel of whole
// views spills 224 and the general form runs twice as long a row: 64 MiB of
// width 8192 less 5 bytes, last segment in the general form 129 us, so 56; 17 rows
// of width 4096 50 against 27.)
#include "fwd_kernel.h"

namespace dwtfrag {

hipError_t launch_fwd_tail(int L, int C1, const void *in, int16_t *pub, int16_t *llout,
                           const StageParams &P, hipStream_t s) {
#define DWTFRAG_CASE(LL, CC) \
  if (L == LL && C1 == CC) return launch_fwd_t<LL, CC, true, true>(in, pub, llout, P, s);
  DWTFRAG_CASE(1, 8) DWTFRAG_CASE(2, 8) DWTFRAG_CASE(3, 8)
  DWTFRAG_CASE(1, 16) DWTFRAG_CASE(2, 16) DWTFRAG_CASE(3, 16) DWTFRAG_CASE(4, 16)
#undef DWTFRAG_CASE
  return hipErrorInvalidValue;
}

}  // namespace dwtfrag
