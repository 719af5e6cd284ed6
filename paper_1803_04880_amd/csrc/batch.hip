// Batches of independent buffers: host planning and the C ABI.
//
// The thesis cuts data into many fixed-size chunks (Ch. 5 section 5.2.1) and
// its GPU runs take many chunks per call.  Here a batch is planned once on the
// host (every item's geometry and launch plan with 16 columns per lane, and
// one queue of tiles per direction, longest first), copied into a caller-owned
// device buffer, where a small kernel writes the tile lists, and then run by
// one persistent launch per direction that drains the direction's queue:
// protect = the forward drain (encryption fused), restore = the inverse drain
// (decryption fused).  The kernels reset their own queue counters when they
// finish, so a direction is one kernel launch and can be captured in a HIP
// graph.
#include "dwtfrag.h"

#include <algorithm>
#include <atomic>
#include <cstring>
#include <memory>
#include <new>
#include <utility>
#include <vector>

#include "batch.h"

namespace dwtfrag {

hipError_t launch_fwd_batch(const BatchItem *items, const int2 *tiles, int64_t n_tiles,
                            BatchCounters *ctr, int blocks, hipStream_t s);
hipError_t launch_inv_batch(const BatchItem *items, const int2 *tiles, int64_t n_tiles,
                            BatchCounters *ctr, int blocks, hipStream_t s);
// The kernels of batches with partial last rows (weak: a build of the planner
// alone for the host has none).
__attribute__((weak)) hipError_t launch_fwd_batch_tail(const BatchItem *items, const int2 *tiles, int64_t n_tiles,
                                                       BatchCounters *ctr, int blocks, hipStream_t s);
__attribute__((weak)) hipError_t launch_inv_batch_tail(const BatchItem *items, const int2 *tiles, int64_t n_tiles,
                                                       BatchCounters *ctr, int blocks, hipStream_t s);
// ... and those of batches of few rows only.
__attribute__((weak)) hipError_t launch_fwd_few_batch(const BatchItem *items, const int2 *tiles, int64_t n_tiles,
                                                      hipStream_t s);
__attribute__((weak)) hipError_t launch_inv_few_batch(const BatchItem *items, const int2 *tiles, int64_t n_tiles,
                                                      unsigned lds, hipStream_t s);
int fwd_batch_blocks_per_cu();
int inv_batch_blocks_per_cu();
int plan_single_stage(uint64_t n, uint32_t width, uint32_t levels, bool forward,
                      const dwtfrag_launch *launch, const AesKey &key, StageParams *P, int *L,
                      int *C1, uint64_t *priv_bytes);

// The tile list of both directions from the queues' runs, a thread per tile;
// the queue counters start at zero (the drains leave them at zero).
__global__ __launch_bounds__(256) void batch_tiles_kernel(const BatchRun *__restrict__ runs, int64_t n_runs,
                                                          int2 *__restrict__ tiles, int64_t n_tiles,
                                                          BatchCounters *__restrict__ ctr) {
  const int64_t t = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (t < n_tiles) tiles[t] = batch_tile(runs, n_runs, t);
  if (t < 2) ctr[t] = BatchCounters{0, 0};
}

}  // namespace dwtfrag

using namespace dwtfrag;

struct dwtfrag_batch {
  uint32_t count = 0;
  std::vector<BatchItem> items;
  std::vector<BatchRun> runs;              // forward queue, then inverse queue
  int64_t n_fwd = 0, n_inv = 0;            // tiles per direction
  int64_t part_fwd = 0, part_inv = 0;      // of them with a partial last row
  bool few_fwd = true, few_inv = true;     // every item is a view of few rows
  unsigned few_lds = 0;                    // LDS of the inverse for them
  int fwd_blocks = 0, inv_blocks = 0;      // persistent grid per direction
  uint64_t off_ctr = 0, off_items = 0, off_runs = 0, off_tiles = 0, bytes = 0;
  char *dev = nullptr;                     // caller's device copy, set by upload
  hipEvent_t uploaded = nullptr;           // the last upload's copies are done
};

namespace {

uint64_t a256(uint64_t v) { return (v + 255) & ~uint64_t(255); }

const dwtfrag_launch *tuned_launch(const dwtfrag_tune_entry *tune, uint32_t n_tune, uint32_t width,
                                   uint32_t levels) {
  for (uint32_t i = 0; i < n_tune; ++i)
    if (tune[i].width == width && tune[i].levels == levels) return &tune[i].launch;
  return nullptr;
}

// Persistent grid of a batch kernel: resident workgroups per CU x CUs.
int persistent_blocks(int per_cu) {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess) dev = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
    cus = 256;
  return cus * std::max(1, per_cu);
}

// Whether a drain runs the kernel whose plain form takes partial last rows.
// The other one runs their tiles in its general form, twice as long a row, at
// the end of a short drain as long again as the drain; this one's checks cost
// every other tile of whole lanes 3 to 20 %.  A few rounds of tiles, where the
// longest tile counts: 30 buffers of 4 to 256 KiB forward / inverse 75 / 91 ->
// 44 / 46 us; longer drains by the share of such tiles: 256 buffers up to 16
// MiB (2 %) 560 / 580 -> 530 / 584, up to 64 MiB (1 %) 1557 / 1595 -> 1522 /
// 1685; 1000 of 100 rows of 4096 (a third of the tiles), four levels, 455 / 561
// -> 405 / 479, and whole 405 / 404 -> 432 / 481.
bool partial_rows_kernel(int64_t part, int64_t tiles, int blocks, int share) {
  return part > 0 && (tiles <= 4 * kWavesPerBlock * int64_t(blocks) || part * share > tiles);
}

// Every item's plans and buffers, and the tiles of each direction counted.
int plan_items(const dwtfrag_item *items, uint32_t count, const dwtfrag_tune_entry *tune,
               uint32_t n_tune, dwtfrag_batch *b) {
  b->count = count;
  b->items.resize(count);
  for (uint32_t i = 0; i < count; ++i) {
    const dwtfrag_item &src = items[i];
    if (!src.in || !src.priv || src.levels == 0 || src.levels > uint32_t(kMaxFused)) return DWTFRAG_EINVAL;
    const auto al16 = [](const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
    if (!al16(src.in) || !al16(src.priv) || !al16(src.pub) || !al16(src.out)) return DWTFRAG_EINVAL;
    // every tile has kBatchCols columns per lane (one kernel serves all depths)
    const dwtfrag_launch *tl = tuned_launch(tune, n_tune, src.width, src.levels);
    if (tl && tl->lane_cols != 0 && tl->lane_cols != 8 && tl->lane_cols != 16) return DWTFRAG_EINVAL;
    const dwtfrag_launch ln{tl ? tl->seg_rows : 0u, uint32_t(kBatchCols)};
    AesKey key;
    expand_key(src.key, src.nonce, &key);
    BatchItem &bi = b->items[i];
    std::memset(&bi, 0, sizeof(bi));
    int Lf = 0, Cf = 0, Li = 0, Ci = 0;
    uint64_t priv_bytes = 0;
    int rc = plan_single_stage(src.n, src.width, src.levels, true, &ln, key, &bi.fwd, &Lf, &Cf, &priv_bytes);
    if (rc == DWTFRAG_OK)
      rc = plan_single_stage(src.n, src.width, src.levels, false, &ln, key, &bi.inv, &Li, &Ci, &priv_bytes);
    if (rc != DWTFRAG_OK) return rc;
    const uint64_t pub_bytes = 2 * (uint64_t(bi.fwd.H) * bi.fwd.W) - priv_bytes;
    if (pub_bytes && !src.pub) return DWTFRAG_EINVAL;
    bi.in = src.in;
    bi.priv = src.priv;
    bi.pub = src.pub;
    bi.out = src.out;
    bi.priv_bytes = priv_bytes;
    bi.levels = int32_t(src.levels);
    b->few_fwd = b->few_fwd && few_rows(bi.fwd, bi.levels, kBatchCols, true);
    b->few_inv = b->few_inv && few_rows(bi.inv, bi.levels, kBatchCols, false);
    if (b->few_inv) b->few_lds = std::max(b->few_lds, inv_few_lds(bi.inv, bi.levels, kBatchCols));
    if (src.n % src.width) {
      b->part_fwd += bi.fwd.n_win;
      b->part_inv += bi.inv.n_win;
    }
    b->n_fwd += bi.fwd.n_waves;
    b->n_inv += bi.inv.n_waves;
    if (b->n_fwd + b->n_inv > 0x7fffffffll) return DWTFRAG_ERANGE;
  }
  return DWTFRAG_OK;
}

// The queues of both directions.  Longest tiles first, so the short tiles of
// small items fill the end of a drain instead of extending it.  A tile's cost
// is the rows it streams (segment plus halos) times the columns of its window:
// one cost per item, so the items are sorted and each one's tiles follow one
// another.  A serving loop plans on its one host thread: 256 MiB at one level,
// 20 Ki tiles a direction, takes 22 us with the upload, where tiles sorted one
// by one and copied whole take 764; and copies of more than 16 KB from
// pageable memory, which tile lists make common, stall a loop for 7 ms now and
// then.
void plan_queues(dwtfrag_batch *b) {
  const auto tile_cost = [](const StageParams &P, int halos) {
    const int64_t seg = int64_t(P.unit_rows) * ((P.units + P.n_seg - 1) / P.n_seg);
    return std::min<int64_t>(P.H, seg + halos * P.halo_b) * std::min(P.W, P.own_w);
  };
  b->runs.reserve(2 * size_t(b->count));
  std::vector<std::pair<int64_t, int>> order(b->count);  // cost, item
  int64_t first = 0;
  for (const auto plan : {&BatchItem::fwd, &BatchItem::inv}) {
    for (uint32_t i = 0; i < b->count; ++i) 
      order[i] = {tile_cost(b->items[i].*plan, plan == &BatchItem::fwd ? 3 : 2), int(i)};
    std::stable_sort(order.begin(), order.end(),
                     [](const auto &x, const auto &y) { return x.first > y.first; });
    for (const auto &o : order) {
      b->runs.push_back({first, o.second, 0});
      first += (b->items[o.second].*plan).n_waves;
    }
  }
}

}  // namespace

extern "C" {

int dwtfrag_batch_create(const dwtfrag_item *items, uint32_t count, const dwtfrag_tune_entry *tune,
                         uint32_t n_tune, dwtfrag_batch **out) {
  if (!out) return DWTFRAG_EINVAL;
  *out = nullptr;
  if (!items || count == 0 || count > (1u << 30) || (n_tune && !tune)) return DWTFRAG_EINVAL;
  std::unique_ptr<dwtfrag_batch> b(new (std::nothrow) dwtfrag_batch());
  if (!b) return DWTFRAG_ERANGE;
  try {
    const int rc = plan_items(items, count, tune, n_tune, b.get());
    if (rc != DWTFRAG_OK) return rc;
    plan_queues(b.get());
  } catch (const std::bad_alloc &) {  // tables larger than the host's memory
    return DWTFRAG_ERANGE;
  }
  b->fwd_blocks = persistent_blocks(fwd_batch_blocks_per_cu());
  b->inv_blocks = persistent_blocks(inv_batch_blocks_per_cu());
  b->off_ctr = 0;
  b->off_items = a256(2 * sizeof(BatchCounters));
  b->off_runs = a256(b->off_items + count * sizeof(BatchItem));
  b->off_tiles = a256(b->off_runs + b->runs.size() * sizeof(BatchRun));
  b->bytes = a256(b->off_tiles + uint64_t(b->n_fwd + b->n_inv) * sizeof(int2));
  *out = b.release();
  return DWTFRAG_OK;
}

uint64_t dwtfrag_batch_device_bytes(const dwtfrag_batch *b) { return b ? b->bytes : 0; }

int dwtfrag_batch_upload(dwtfrag_batch *b, void *device_plan, uint64_t device_bytes, void *stream) {
  if (!b || !device_plan || (reinterpret_cast<uintptr_t>(device_plan) & 255)) return DWTFRAG_EINVAL;
  if (device_bytes < b->bytes) return DWTFRAG_EWORKSPACE;
  char *dev = static_cast<char *>(device_plan);
  hipStream_t st = static_cast<hipStream_t>(stream);
  // The copies run asynchronously on the stream: their sources (the plan's own
  // tables) stay in place until dwtfrag_batch_destroy, which waits for the
  // event recorded behind them.
  if (hipMemcpyAsync(dev + b->off_items, b->items.data(), b->items.size() * sizeof(BatchItem),
                     hipMemcpyHostToDevice, st) != hipSuccess)
    return DWTFRAG_EDEVICE;
  if (hipMemcpyAsync(dev + b->off_runs, b->runs.data(), b->runs.size() * sizeof(BatchRun),
                     hipMemcpyHostToDevice, st) != hipSuccess)
    return DWTFRAG_EDEVICE;
  const int64_t n_tiles = b->n_fwd + b->n_inv;
  hipLaunchKernelGGL(batch_tiles_kernel, dim3(unsigned((n_tiles + 255) / 256)), dim3(256), 0, st,
                     reinterpret_cast<const BatchRun *>(dev + b->off_runs), int64_t(b->runs.size()),
                     reinterpret_cast<int2 *>(dev + b->off_tiles), n_tiles,
                     reinterpret_cast<BatchCounters *>(dev + b->off_ctr));
  if (hipGetLastError() != hipSuccess) return DWTFRAG_EDEVICE;
  if (!b->uploaded && hipEventCreateWithFlags(&b->uploaded, hipEventDisableTiming) != hipSuccess) {
    b->uploaded = nullptr;
    return DWTFRAG_EDEVICE;
  }
  if (hipEventRecord(b->uploaded, st) != hipSuccess) return DWTFRAG_EDEVICE;
  b->dev = dev;
  return DWTFRAG_OK;
}

int dwtfrag_batch_protect(const dwtfrag_batch *b, void *stream) {
  if (!b || !b->dev) return DWTFRAG_EINVAL;
  if (b->n_fwd == 0) return DWTFRAG_OK;
  BatchCounters *ctr = reinterpret_cast<BatchCounters *>(b->dev + b->off_ctr);
  const BatchItem *items = reinterpret_cast<const BatchItem *>(b->dev + b->off_items);
  const int2 *tiles = reinterpret_cast<const int2 *>(b->dev + b->off_tiles);
  if (b->few_fwd && launch_fwd_few_batch && b->n_fwd <= kMaxLaunchWaves)
    return launch_fwd_few_batch(items, tiles, b->n_fwd, static_cast<hipStream_t>(stream)) == hipSuccess
               ? DWTFRAG_OK : DWTFRAG_EDEVICE;
  const int blocks = int(std::min<int64_t>(b->fwd_blocks, (b->n_fwd + kWavesPerBlock - 1) / kWavesPerBlock));
  const auto launch = launch_fwd_batch_tail && partial_rows_kernel(b->part_fwd, b->n_fwd, b->fwd_blocks, 200)
                          ? launch_fwd_batch_tail : launch_fwd_batch;
  if (launch(items, tiles, b->n_fwd, ctr, blocks, static_cast<hipStream_t>(stream)) != hipSuccess)
    return DWTFRAG_EDEVICE;
  return DWTFRAG_OK;
}

int dwtfrag_batch_restore(const dwtfrag_batch *b, void *stream) {
  if (!b || !b->dev) return DWTFRAG_EINVAL;
  for (const BatchItem &i : b->items)
    if (!i.out) return DWTFRAG_EINVAL;
  if (b->n_inv == 0) return DWTFRAG_OK;
  BatchCounters *ctr = reinterpret_cast<BatchCounters *>(b->dev + b->off_ctr) + 1;
  const BatchItem *items = reinterpret_cast<const BatchItem *>(b->dev + b->off_items);
  const int2 *tiles = reinterpret_cast<const int2 *>(b->dev + b->off_tiles) + b->n_fwd;
  if (b->few_inv && launch_inv_few_batch && b->n_inv <= kMaxLaunchWaves)
    return launch_inv_few_batch(items, tiles, b->n_inv, b->few_lds, static_cast<hipStream_t>(stream)) == hipSuccess
               ? DWTFRAG_OK : DWTFRAG_EDEVICE;
  const int blocks = int(std::min<int64_t>(b->inv_blocks, (b->n_inv + kWavesPerBlock - 1) / kWavesPerBlock));
  const auto launch = launch_inv_batch_tail && partial_rows_kernel(b->part_inv, b->n_inv, b->inv_blocks, 20)
                          ? launch_inv_batch_tail : launch_inv_batch;
  if (launch(items, tiles, b->n_inv, ctr, blocks, static_cast<hipStream_t>(stream)) != hipSuccess)
    return DWTFRAG_EDEVICE;
  return DWTFRAG_OK;
}

void dwtfrag_batch_destroy(dwtfrag_batch *b) {
  if (!b) return;
  if (b->uploaded) {  // the copies read the plan's tables until then
    hipEventSynchronize(b->uploaded);
    hipEventDestroy(b->uploaded);
  }
  delete b;
}

}  // extern "C"
