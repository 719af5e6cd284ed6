// Host check that launches are planned for the device's own size: with fewer
// compute units, as a partition has, the segments of an image grow in both
// directions and the grid shrinks with the units; with 256 they are those that
// the launch rules were measured at.  Built from api.hip for the host only,
// with the device queries replaced.
#include <cstdint>
#include <cstdio>

#include "dwtfrag.h"
#include "common.h"

static int device = 0;
static const int units[] = {256, 128, 64, 32};
static int waves[2];

extern "C" {
hipError_t hipGetDeviceCount(int *n) { *n = 4; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = device; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int d) { *v = units[d]; return hipSuccess; }
}
namespace dwtfrag {
hipError_t launch_fwd(int, int, bool, const void *, int16_t *, int16_t *, const StageParams &P,
                      hipStream_t) { waves[0] = P.n_waves; return hipSuccess; }
hipError_t launch_inv(int, int, bool, const int16_t *, const int16_t *, void *, const StageParams &P,
                      hipStream_t) { waves[1] = P.n_waves; return hipSuccess; }
hipError_t launch_ctr(const uint8_t *, uint8_t *, uint64_t, const AesKey &, uint64_t, hipStream_t) {
  return hipErrorInvalidValue;
}
}  // namespace dwtfrag

int main() {
  int failures = 0;
  const uint8_t key[16] = {0};
  uint8_t *p = reinterpret_cast<uint8_t *>(uintptr_t(1) << 20);
  int16_t *q = reinterpret_cast<int16_t *>(uintptr_t(1) << 20);
  const uint64_t n = 1 << 22;
  int first[2] = {0, 0}, before[2] = {0, 0};
  for (device = 0; device < 4; ++device) {
    for (int again = 0; again < 2; ++again) {  // the second from what is kept
      if (dwtfrag_protect(p, n, 2048, 3, key, key, p, q, nullptr, 0, nullptr, nullptr) != DWTFRAG_OK ||
          dwtfrag_restore(p, q, n, 2048, 3, key, key, p, nullptr, 0, nullptr, nullptr) != DWTFRAG_OK)
        return 2;
      std::printf("%d units: %d forward, %d inverse wavefronts\n", units[device], waves[0], waves[1]);
      for (int d = 0; d < 2; ++d) {
        if (device == 0) first[d] = before[d] = waves[d];
        else if (!again && !(waves[d] < before[d])) ++failures;
        if (again && waves[d] != before[d]) ++failures;
        before[d] = waves[d];
      }
    }
  }
  // (6 windows of 16-row segments, 5 of 8-row ones)
  if (first[0] != 6 * 128 || first[1] != 5 * 256) ++failures;
  std::printf("%d failures\n", failures);
  return failures != 0;
}
