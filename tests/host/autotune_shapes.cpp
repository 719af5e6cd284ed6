// Host check of the launch shapes that dwtfrag_autotune times: no two give the
// same launches except the default's own, the default is among them, heights
// below 64 rows are, and the shape that it returns is the one whose launches
// were the fastest.  Built from api.hip for the host only: the launchers below
// record the plans, and the events report a time made from them.
#include <cstdint>
#include <cstdio>
#include <map>
#include <set>
#include <string>

#include "dwtfrag.h"
#include "common.h"

static std::string pass;             // the launches since the last event
static std::set<std::string> seen;   // of every timed pass
static std::map<std::string, float> cost;
static std::string timed;

static hipError_t note(char way, int L, int C1, const dwtfrag::StageParams &P) {
  pass += way + std::to_string(L) + "x" + std::to_string(C1) + ":" + std::to_string(P.n_seg) + "/" +
          std::to_string(P.n_win) + " ";
  return hipSuccess;
}
namespace dwtfrag {
hipError_t launch_fwd(int L, int C1, bool, const void *, int16_t *, int16_t *, const StageParams &P,
                      hipStream_t) { return note('f', L, C1, P); }
hipError_t launch_inv(int L, int C1, bool, const int16_t *, const int16_t *, void *, const StageParams &P,
                      hipStream_t) { return note('i', L, C1, P); }
hipError_t launch_ctr(const uint8_t *, uint8_t *, uint64_t, const AesKey &, uint64_t, hipStream_t) {
  return hipErrorInvalidValue;
}
}  // namespace dwtfrag

extern "C" {
hipError_t hipEventCreate(hipEvent_t *e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
static int records = 0;
hipError_t hipEventRecord(hipEvent_t, hipStream_t) {
  if (records++ % 2 == 0) pass.clear();
  else timed = pass;
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
  *ms = cost.count(timed) ? cost[timed] : 10.0f;
  seen.insert(timed);
  return hipSuccess;
}
}

static std::string launches_of(uint64_t n, uint32_t w, uint32_t L, const dwtfrag_launch *ln, uint64_t ws) {
  const uint8_t key[16] = {0};
  uint8_t *p = reinterpret_cast<uint8_t *>(uintptr_t(1) << 20);
  pass.clear();
  if (dwtfrag_protect(p, n, w, L, key, key, p, reinterpret_cast<int16_t *>(p), p, ws, ln, nullptr) != DWTFRAG_OK ||
      dwtfrag_restore(p, reinterpret_cast<int16_t *>(p), n, w, L, key, key, p, p, ws, ln, nullptr) != DWTFRAG_OK)
    return "failed";
  return pass;
}

int main() {
  int failures = 0;
  const struct { uint64_t n; uint32_t w, L; } calls[] = {
      {1 << 18, 512, 1}, {1 << 24, 4096, 1}, {1 << 24, 4096, 2}, {1 << 24, 4096, 3}, {1 << 24, 4096, 4},
      {1 << 28, 32768, 3}, {12000017, 3001, 2}, {1 << 26, 8192, 6}, {1 << 26, 8192, 8}, {30000, 5000, 2}};
  for (const auto &c : calls) {
    dwtfrag_geom g;
    if (dwtfrag_geometry(c.n, c.w, c.L, &g) != DWTFRAG_OK) return 2;
    void *scratch = reinterpret_cast<void *>(uintptr_t(1) << 22);
    const uint8_t *in = reinterpret_cast<const uint8_t *>(uintptr_t(1) << 20);
    const uint64_t bytes = uint64_t(1) << 40;
    dwtfrag_launch best{9, 9};
    float us = 0;
    seen.clear();
    cost.clear();
    records = 0;
    if (dwtfrag_autotune(in, c.n, c.w, c.L, scratch, bytes, 1, &best, &us, nullptr) != DWTFRAG_OK) ++failures;
    const int timed_passes = records / 2;
    const std::string def = launches_of(c.n, c.w, c.L, nullptr, g.workspace_bytes);
    if (!seen.count(def)) { std::printf("the default is not timed\n"); ++failures; }
    if (int(seen.size()) + 2 < timed_passes) {  // (the default may be one of the heights, in each column count)
      std::printf("%d passes, %zu shapes\n", timed_passes, seen.size());
      ++failures;
    }
    const auto shapes = seen;
    for (const auto &s : shapes) {  // each in turn the fastest
      cost.clear();
      cost[s] = 1.0f;
      records = 0;
      if (dwtfrag_autotune(in, c.n, c.w, c.L, scratch, bytes, 1, &best, &us, nullptr) != DWTFRAG_OK ||
          launches_of(c.n, c.w, c.L, &best, g.workspace_bytes) != s || us != 1000.0f) {
        std::printf("shape {%u, %u} returned for %s\n", best.seg_rows, best.lane_cols, s.c_str());
        ++failures;
      }
    }
    bool low = g.height <= 64;
    for (uint32_t r = 8; r < 64 && !low; r += 8) {
      const dwtfrag_launch ln{r, uint32_t(c.L >= 4 ? 16 : 8)};
      low = r % (1u << (c.L < 4 ? c.L : 4)) == 0 && seen.count(launches_of(c.n, c.w, c.L, &ln, g.workspace_bytes));
    }
    if (!low) { std::printf("no height below 64 rows\n"); ++failures; }
    std::printf("%llu bytes, width %u, %u levels: %d passes, %zu shapes\n", (unsigned long long)c.n, c.w, c.L,
                timed_passes, shapes.size());
  }
  std::printf("%d failures\n", failures);
  return failures != 0;
}
