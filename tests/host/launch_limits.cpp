// Host check of the launches that protect and restore plan: over every
// accepted height, narrow and ordinary widths, depths and launch shapes, a
// launch has fewer than the 2^32 work-items that HIP takes per dimension, and
// no segment has more low rows than a wavefront keeps the keystream of.  Built
// from api.hip for the host only; the launchers below record the plan and
// report success, so that every stage of a call is seen.
#include <algorithm>
#include <cstdint>
#include <cstdio>

#include "dwtfrag.h"
#include "common.h"

static long launches = 0, failures = 0;
static const char *what = "";

static hipError_t planned(int L, int C1, const dwtfrag::StageParams &P) {
  using namespace dwtfrag;
  const int per = block_waves(P.n_waves, 256);
  const uint64_t threads = (uint64_t(P.n_waves) + per - 1) / per * per * 64;
  const int64_t most_units = (int64_t(P.units) + P.n_seg - 1) / P.n_seg;
  const bool ok = P.n_waves > 0 && P.n_waves == int64_t(P.n_win) * P.n_seg && threads < (uint64_t(1) << 32) &&
                  most_units <= fwd_ll_rows(L, C1) && (C1 == 8 || C1 == 16) && (L < 4 || C1 == 16);
  ++launches;
  if (!ok && ++failures < 20)
    std::printf("%s: %d levels, %d columns a lane, %d x %d: %d wavefronts, %llu work-items, %lld units a segment\n",
                what, L, C1, P.H, P.W, P.n_waves, (unsigned long long)threads, (long long)most_units);
  return ok ? hipSuccess : hipErrorInvalidConfiguration;
}

namespace dwtfrag {
hipError_t launch_fwd(int L, int C1, bool, const void *, int16_t *, int16_t *, const StageParams &P,
                      hipStream_t) { return planned(L, C1, P); }
hipError_t launch_inv(int L, int C1, bool, const int16_t *, const int16_t *, void *, const StageParams &P,
                      hipStream_t) { return planned(L, C1, P); }
hipError_t launch_ctr(const uint8_t *, uint8_t *, uint64_t, const AesKey &, uint64_t, hipStream_t) {
  return hipErrorInvalidValue;
}
}  // namespace dwtfrag

int main() {
  const uint8_t key[16] = {1}, nonce[16] = {2};
  uint8_t *fp = reinterpret_cast<uint8_t *>(uintptr_t(1) << 20);
  int16_t *fq = reinterpret_cast<int16_t *>(uintptr_t(1) << 21);
  const uint64_t heights[] = {1, 2, 47, 512, 100003, uint64_t(1) << 26, (uint64_t(1) << 30) - 1, (uint64_t(1) << 30) + 1,
                              1610612737, 1700000000, 0x7FFF0000ull - 1, 0x7FFF0000ull};
  const uint32_t widths[] = {1, 2, 3, 8, 16, 100, 384, 512, 513, 1024, 1025, 4096, 32768, 1u << 20};
  const dwtfrag_launch shapes[] = {{0, 0}, {0, 8}, {0, 16}, {1, 8}, {1, 16}, {64, 8}, {64, 16}, {256, 16}, {1000000, 8}};
  for (uint64_t h : heights)
    for (uint32_t w : widths)
      for (uint32_t L : {1u, 2u, 3u, 4u, 5u, 6u, 7u, 9u})
        for (const dwtfrag_launch &ln : shapes) {
          const uint64_t n = h * w;
          if (3 * n > uint64_t(288) << 30) continue;  // bytes and fragments beyond the device's memory
          dwtfrag_geom g;
          if (dwtfrag_geometry(n, w, L, &g) != DWTFRAG_OK) {
            ++failures;
            continue;
          }
          char buf[128];
          std::snprintf(buf, sizeof(buf), "%llu rows of %u, %u levels, shape {%u, %u}", (unsigned long long)h, w, L,
                        ln.seg_rows, ln.lane_cols);
          what = buf;
          if (dwtfrag_protect(fp, n, w, L, key, nonce, fp, fq, fp, g.workspace_bytes, &ln, nullptr) != DWTFRAG_OK ||
              dwtfrag_restore(fp, fq, n, w, L, key, nonce, fp, fp, g.workspace_bytes, &ln, nullptr) != DWTFRAG_OK)
            ++failures;
        }
  std::printf("%ld launches, %ld failures\n", launches, failures);
  return failures != 0;
}
