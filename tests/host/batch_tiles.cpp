// Host check of a batch's tile lists: each direction's list holds every tile
// of every item once, in the order of a stable sort of all tiles by cost,
// longest first; and planning a buffer of many tiles takes a fraction of the
// time of that sort, and its tables a fraction of the list's bytes.  Includes the planner's source to see its tables.
#include "batch.hip"

#include <chrono>
#include <cstdio>

namespace dwtfrag {
hipError_t launch_fwd(int, int, bool, const void *, int16_t *, int16_t *, const StageParams &,
                      hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_inv(int, int, bool, const int16_t *, const int16_t *, void *, const StageParams &,
                      hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_ctr(const uint8_t *, uint8_t *, uint64_t, const AesKey &, uint64_t,
                      hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_fwd_batch(const BatchItem *, const int2 *, int64_t, BatchCounters *, int,
                            hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_inv_batch(const BatchItem *, const int2 *, int64_t, BatchCounters *, int,
                            hipStream_t) { return hipErrorInvalidValue; }
int fwd_batch_blocks_per_cu() { return 2; }
int inv_batch_blocks_per_cu() { return 2; }
}  // namespace dwtfrag

static int64_t cost(const StageParams &P, bool forward) {
  const int64_t seg = int64_t(P.unit_rows) * ((P.units + P.n_seg - 1) / P.n_seg);
  return std::min<int64_t>(P.H, seg + (forward ? 3 : 2) * P.halo_b) * std::min(P.W, P.own_w);
}

static std::vector<int2> sorted_tiles(const dwtfrag_batch &b, StageParams BatchItem::*plan) {
  std::vector<int2> t;
  for (uint32_t i = 0; i < b.count; ++i)
    for (int w = 0; w < (b.items[i].*plan).n_waves; ++w) t.push_back(make_int2(int(i), w));
  std::vector<int64_t> c(b.count);
  for (uint32_t i = 0; i < b.count; ++i) c[i] = cost(b.items[i].*plan, plan == &BatchItem::fwd);
  std::stable_sort(t.begin(), t.end(), [&](const int2 &x, const int2 &y) { return c[x.x] > c[y.x]; });
  return t;
}

static dwtfrag_item item(uint64_t n, uint32_t levels) {
  dwtfrag_item it{};
  it.in = reinterpret_cast<const uint8_t *>(uintptr_t(1) << 20);
  it.out = reinterpret_cast<uint8_t *>(uintptr_t(1) << 20);
  it.priv = reinterpret_cast<uint8_t *>(uintptr_t(1) << 20);
  it.pub = reinterpret_cast<int16_t *>(uintptr_t(1) << 21);
  it.n = n;
  it.width = dwtfrag_default_width(n);
  it.levels = levels;
  return it;
}

template <class F> static double best_us(const F &f) {
  double best = 1e30;
  for (int k = 0; k < 15; ++k) {
    const auto t0 = std::chrono::steady_clock::now();
    f();
    best = std::min(best, std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count());
  }
  return best;
}

int main() {
  int failures = 0;
  std::vector<dwtfrag_item> items;
  uint64_t r = 12345;
  for (int i = 0; i < 200; ++i) {  // sizes of several costs, many of them equal
    r = r * 6364136223846793005ull + 1442695040888963407ull;
    items.push_back(item((uint64_t(1) << (12 + (r >> 60))) + (r >> 40) % 3 * 4000, 1 + uint32_t((r >> 33) & 3)));
  }
  for (size_t count : {size_t(1), size_t(2), size_t(37), items.size()}) {
    dwtfrag_batch *b = nullptr;
    if (dwtfrag_batch_create(items.data(), uint32_t(count), nullptr, 0, &b) != DWTFRAG_OK) return 2;
    auto want = sorted_tiles(*b, &BatchItem::fwd);
    const auto inv = sorted_tiles(*b, &BatchItem::inv);
    const bool sizes = b->n_fwd == int64_t(want.size()) && b->n_inv == int64_t(inv.size());
    want.insert(want.end(), inv.begin(), inv.end());
    bool same = sizes;
    for (size_t k = 0; same && k < want.size(); ++k) {  // as batch_tiles_kernel writes them
      const int2 t = batch_tile(b->runs.data(), int64_t(b->runs.size()), int64_t(k));
      same = want[k].x == t.x && want[k].y == t.y;
    }
    if (!same) {
      std::printf("%zu items: the lists differ from the sorted tiles\n", count);
      ++failures;
    }
    dwtfrag_batch_destroy(b);
  }
  const dwtfrag_item large = item(uint64_t(1) << 28, 1);
  const double plan = best_us([&] {
    dwtfrag_batch *b = nullptr;
    if (dwtfrag_batch_create(&large, 1, nullptr, 0, &b) == DWTFRAG_OK) dwtfrag_batch_destroy(b);
  });
  dwtfrag_batch *b = nullptr;
  if (dwtfrag_batch_create(&large, 1, nullptr, 0, &b) != DWTFRAG_OK) return 2;
  size_t total = 0;
  const double sort = best_us([&] { total = sorted_tiles(*b, &BatchItem::fwd).size() + sorted_tiles(*b, &BatchItem::inv).size(); });
  const size_t copied = b->items.size() * sizeof(BatchItem) + b->runs.size() * sizeof(BatchRun);
  if (copied > total * sizeof(int2) / 10) ++failures;
  dwtfrag_batch_destroy(b);
  std::printf("256 MiB, one level: planned in %.0f us; sorting its %zu tiles %.0f us\n", plan, total, sort);
  if (plan > 0.5 * sort) ++failures;
  std::printf("%d failures\n", failures);
  return failures != 0;
}
