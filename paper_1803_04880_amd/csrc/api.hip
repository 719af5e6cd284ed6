// C ABI of the library: validation, geometry, AES key schedule, stage and
// launch planning.  Declarations and contracts are in include/dwtfrag.h.
#include "dwtfrag.h"

#include <algorithm>
#include <cstring>
#include <mutex>

#include "common.h"

namespace dwtfrag {

hipError_t launch_fwd(int L, int C1, bool u8in, const void *in, int16_t *pub, int16_t *llout,
                      const StageParams &P, hipStream_t s);
hipError_t launch_inv(int L, int C1, bool u8out, const int16_t *llin, const int16_t *pub,
                      void *out, const StageParams &P, hipStream_t s);
hipError_t launch_ctr(const uint8_t *in, uint8_t *out, uint64_t nbytes, const AesKey &key,
                      uint64_t first_block, hipStream_t s);

static constexpr AesTables kHostTables = make_aes_tables();

void expand_key(const uint8_t key[16], const uint8_t nonce[16], AesKey *out) {
  // FIPS-197 key expansion, Nk = 4, Nr = 10.  Words are kept little-endian
  // (byte 0 of a word in bits 0..7), matching the device state layout.
  uint32_t *w = out->rk;
  for (int i = 0; i < 4; ++i)
    w[i] = uint32_t(key[4 * i]) | (uint32_t(key[4 * i + 1]) << 8) |
           (uint32_t(key[4 * i + 2]) << 16) | (uint32_t(key[4 * i + 3]) << 24);
  uint8_t rcon = 1;
  for (int i = 4; i < 44; ++i) {
    uint32_t t = w[i - 1];
    if (i % 4 == 0) {
      t = (t >> 8) | (t << 24);  // RotWord on bytes (a0 a1 a2 a3) -> (a1 a2 a3 a0)
      t = uint32_t(kHostTables.sbox[t & 0xFF]) | (uint32_t(kHostTables.sbox[(t >> 8) & 0xFF]) << 8) |
          (uint32_t(kHostTables.sbox[(t >> 16) & 0xFF]) << 16) |
          (uint32_t(kHostTables.sbox[t >> 24]) << 24);
      t ^= rcon;
      rcon = gf_mul(rcon, 2);
    }
    w[i] = w[i - 4] ^ t;
  }
  uint64_t hi = 0, lo = 0;
  for (int i = 0; i < 8; ++i) {
    hi = (hi << 8) | nonce[i];
    lo = (lo << 8) | nonce[8 + i];
  }
  out->nonce_hi = hi;
  out->nonce_lo = lo;
}

namespace {

// Compute units of every device, asked once; 256 where a query fails (no
// device: planning only).
struct DeviceUnits {
  static constexpr int kDev = 64;
  int units[kDev];
  bool same = true;  // all devices alike: the current one need not be asked for
  DeviceUnits() {
    int count = 0;
    if (hipGetDeviceCount(&count) != hipSuccess) count = 0;
    for (int d = 0; d < kDev; ++d) {
      units[d] = 256;
      int n = 0;
      if (d < count && hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, d) == hipSuccess && n > 0)
        units[d] = n;
      if (d < count && units[d] != units[0]) same = false;
    }
    if (count > kDev) same = false;
  }
};

}  // namespace

int device_cus() {
  static const DeviceUnits all;
  if (all.same) return all.units[0];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= DeviceUnits::kDev) return 256;
  return all.units[dev];
}

namespace {

// Bytes of the static workspace behind dwtfrag_protect_noalloc (16 MiB).
constexpr uint64_t kScratchBytes = uint64_t(16) << 20;

// Deepest decomposition accepted, and the fused stages it takes.  Geometry and
// launch plans live in fixed arrays of these sizes, so planning a call
// allocates nothing, on the host or the device.
constexpr uint32_t kMaxLevels = 32;
constexpr int kMaxStages = int((kMaxLevels + kMaxFused - 1) / kMaxFused);

struct Geometry {
  uint64_t n;
  uint32_t W, H, levels;
  uint64_t h[kMaxLevels + 1], w[kMaxLevels + 1];  // level dims 0..levels
  uint64_t priv_bytes, pub_bytes, ws_bytes;
  uint64_t ws_off[kMaxStages];  // workspace byte offset of LL_{4(s+1)}, s = 0..stages-2
  int stages;
};

uint64_t align256(uint64_t v) { return (v + 255) & ~uint64_t(255); }

int make_geometry(uint64_t n, uint32_t width, uint32_t levels, Geometry *g) {
  if (n == 0 || width == 0 || levels == 0 || levels > kMaxLevels) return DWTFRAG_EINVAL;
  if (width > uint32_t(kMaxDim)) return DWTFRAG_ERANGE;
  const uint64_t H = (n + width - 1) / width;
  if (H > uint64_t(kMaxDim)) return DWTFRAG_ERANGE;
  if (H * uint64_t(width) > (uint64_t(1) << 62)) return DWTFRAG_ERANGE;
  g->n = n;
  g->W = width;
  g->H = uint32_t(H);
  g->levels = levels;
  std::memset(g->h, 0, sizeof(g->h));
  std::memset(g->w, 0, sizeof(g->w));
  std::memset(g->ws_off, 0, sizeof(g->ws_off));
  g->h[0] = H;
  g->w[0] = width;
  for (uint32_t l = 1; l <= levels; ++l) {
    g->h[l] = (g->h[l - 1] + 1) / 2;
    g->w[l] = (g->w[l - 1] + 1) / 2;
  }
  const uint64_t ll = g->h[levels] * g->w[levels];
  g->priv_bytes = 2 * ll;
  g->pub_bytes = 2 * (H * width - ll);
  g->stages = int((levels + kMaxFused - 1) / kMaxFused);
  uint64_t ws = 0;
  for (int s = 0; s + 1 < g->stages; ++s) {
    g->ws_off[s] = ws;
    const int lv = kMaxFused * (s + 1);
    ws += align256(2 * g->h[lv] * g->w[lv]);
  }
  g->ws_bytes = ws;
  return DWTFRAG_OK;
}

// Element offset in pub of level l's three bands (levels stored coarsest
// first: L, L-1, ..., 1).
void level_offsets(const Geometry &g, uint32_t l, int64_t *hl, int64_t *lh, int64_t *hh) {
  uint64_t off = 0;
  for (uint32_t m = g.levels; m > l; --m) off += g.h[m - 1] * g.w[m - 1] - g.h[m] * g.w[m];
  *hl = int64_t(off);
  *lh = int64_t(off + g.h[l] * (g.w[l - 1] - g.w[l]));
  *hh = int64_t(off + g.h[l] * (g.w[l - 1] - g.w[l]) + (g.h[l - 1] - g.h[l]) * g.w[l]);
}

int round_up(int v, int m) { return (v + m - 1) / m * m; }

// Rows of a forward segment.  A segment recomputes 2^(L+1) + 2^L - 3 rows, so
// taller is less work, but every wavefront is one serial stream: a launch of
// its own wants about 940 of them on 256 compute units (at one level, where
// the cipher counts most, 1536) before its segments grow past one unit.  The
// tallest worth it, by level (measured, us at 4096 columns, 16 / 64 MiB, or
// 32768, 256 MiB):
//   1: 24 rows 24.9 / 68.6 / 228 (8: 25.0 / 67.9 / 252);
//   2: 16 rows 16.6 / 44.8 / 179, 32: 19.5 / 46.7 / 168;
//   3: 96 rows (8 columns a lane) 46.9 at 64 MiB, 48: 47.7, 16: 56.2; at 16
//      columns 24 rows 176 at 256 MiB (32: 182, 96: 208);
//   4: 96 rows 53.7 at 64 MiB (64: 60.9), 64 rows 198 at 256 MiB (96: 214).
int fwd_seg_rows(int L, int C1, int n_win, int H, uint64_t cells, int cus) {
  const bool large = cells >= (uint64_t(1) << 27);
  const int most = L == 1 ? 24 : L == 2 ? (large ? 32 : 16) : L == 3 ? (C1 == 16 ? 24 : 96) : large ? 64 : 96;
  const int64_t want = int64_t(n_win) * H * 256 / (int64_t(L == 1 ? 1536 : 940) * cus);
  const int rows = round_up(int(std::min<int64_t>(std::max<int64_t>(want, 1), most)), 1 << L);
  return std::min(rows, fwd_max_rows(L, C1));
}

// Rows of an inverse segment: the least that make no more than two wavefronts
// for each SIMD, of which a compute unit has four (four wavefronts where the
// row's end cuts a lane's columns: those take 2.5 times as long a row), up to
// 32 rows (at four levels 48).  Measured on 256 units, us: 16 MiB of width 4096 at three levels 24 rows
// 17.7, 16: 19.0, 32: 20.0; 12 MB of width 3001 at two levels 8 rows 23.9,
// 16: 26.4, 32: 32.3; 256 MiB at three levels 32 rows 161, 24: 162, 48: 163,
// 16: 176; 64 MiB at four levels 48 rows 57.3, 32: 58.6, 64: 66.5.
int inv_seg_rows(int L, int C1, int n_win, int W, int H, int cus) {
  const int unit = 1 << L, most = std::min(L == 4 ? 48 : 32, inv_max_rows(L, C1));
  const int64_t waves = int64_t(W % C1 ? 16 : 8) * cus;
  int rows = unit;
  while (rows < most && int64_t(n_win) * ((H + rows - 1) / rows) > waves) rows += unit;
  return std::min(rows, most);
}

// Rows of a batch item's tiles.  The items share the device, so that no tile
// need be short to fill it: 256 items of 4 KiB to 64 MiB, 1.8 GB, forward /
// inverse, 24 rows 1458 / 1451 us, 32: 1396 / 1368, 48: 1361 / 1357, 64: 1373
// / 1388, 96: 1378 / 1417; as single launches' 1562 / 1372.
constexpr int kBatchRows = 48;

// Whether a stage runs at 16 columns a lane by default: 8 but 16 (the per-row
// work spread over twice the columns) for a forward of three levels and 128 Mi
// elements (176 against 181 us at 256 MiB; 46.2 against 46.9 at 64 MiB, and one
// and two levels are as fast at 8: 228, 168 against 227, 169).  The inverse at
// 16 is slower at all sizes (256 MiB at one, two and three levels 268, 166, 161
// against 253, 162, 158 us).  Four levels need 16 columns.
bool wide_stage(bool forward, int L, uint64_t cells) {
  return L == 4 || (forward && L == 3 && cells >= (uint64_t(1) << 27));
}

// Fill stage s's parameters.  forward selects the halo shape of the direction;
// alone: the stage runs as its own launch (not as one item of a batch that
// shares the device).
int plan_stage(const Geometry &g, int s, bool forward, const dwtfrag_launch *launch,
               const AesKey &key, StageParams *P, int *L_out, int *C1_out, bool alone) {
  std::memset(P, 0, sizeof(*P));
  const int lv0 = kMaxFused * s;  // global level of the stage input
  const int L = int(std::min<uint32_t>(kMaxFused, g.levels - lv0));
  const uint64_t cells = uint64_t(g.h[lv0]) * g.w[lv0];
  int C1 = (launch && launch->lane_cols) ? int(launch->lane_cols) : wide_stage(forward, L, cells) ? 16 : 8;
  if (C1 != 8 && C1 != 16) return DWTFRAG_EINVAL;
  if (L == 4) C1 = 16;
  // (a launch of more than 2^30 rows: 16 columns' segments would be too many)
  if (alone && L == 1 && g.h[lv0] / fwd_max_rows(L, C1) >= uint64_t(kMaxLaunchWaves)) C1 = 8;
  P->H = int32_t(g.h[lv0]);
  P->W = int32_t(g.w[lv0]);
  P->n_valid = (s == 0) ? int64_t(g.n) : int64_t(g.h[lv0] * g.w[lv0]);
  for (int l = 0; l <= L; ++l) {
    P->hdim[l] = int32_t(g.h[lv0 + l]);
    P->wdim[l] = int32_t(g.w[lv0 + l]);
  }
  for (int l = 1; l <= L; ++l)
    level_offsets(g, uint32_t(lv0 + l), &P->off_hl[l], &P->off_lh[l], &P->off_hh[l]);
  // halos (level-0 samples of this stage): forward needs 2^(L+1)-2 before and
  // 2^L-1 after an owned range, inverse the reverse; rows are streamed with
  // 2^(L+1) / 2^L (forward) and 2^L / 2^L (inverse) extra rows.
  const int big = (1 << (L + 1)) - 2, small = (1 << L) - 1;
  const int hl = round_up(forward ? big : small, C1);
  const int hr = round_up(forward ? small : big, C1);
  const int span = 64 * C1;
  if (P->W <= span) {
    P->own_w = P->W;
    P->n_win = 1;
  } else {
    P->own_w = span - hl - hr;
    // A window owns whole lines of what it writes: lines that two windows
    // share are written in parts.  Forward: 128 bytes of its level-1 band rows
    // (three levels at 8 columns a lane, 384 / 448 / 480 / 488 of 512 columns
    // owned, us: 4 MiB 13.2 / 12.9 / 13.1 / 13.1, 16 MiB 19.1 / 19.4 / 18.2 /
    // 18.1, 64 MiB 47.8 / 51.1 / 56.0 / 60.2, 256 MiB 157 / 174 / 203 / 227; two
    // levels 16 MiB 16.2 / 16.8 / 18.0 / 20.9, 256 MiB 152 / 154 / 181 / 194).
    // Inverse: 64 bytes of an output row (256 MiB at three levels: 448 columns
    // 165 us, 488: 172, 384: 170, each before rows loaded ahead were clamped),
    // but at one level, where the cipher of the columns that windows share costs
    // more, all it can (496 columns 253 us, 448: 276).
    const int whole = forward ? 128 : L == 1 ? 1 : 64;
    P->own_w = P->own_w / whole * whole;
    P->n_win = (P->W + P->own_w - 1) / P->own_w;
  }
  P->halo_l = hl;
  P->halo_b = 1 << L;
  const int unit = 1 << L;
  P->unit_rows = unit;
  P->units = (P->H + unit - 1) / unit;
  const int cus = alone ? device_cus() : 256;
  int rows = !alone    ? kBatchRows
             : forward ? fwd_seg_rows(L, C1, P->n_win, P->H, cells, cus)
                       : inv_seg_rows(L, C1, P->n_win, P->W, P->H, cus);
  if (launch && launch->seg_rows)
    rows = std::max(unit, round_up(int(std::min<uint32_t>(launch->seg_rows, uint32_t(P->H))), unit));
  const int most = forward ? fwd_max_rows(L, C1) : inv_max_rows(L, C1);
  rows = std::min(rows, most);
  if (alone && int64_t(P->n_win) * ((P->H + rows - 1) / rows) > kMaxLaunchWaves) rows = most;
  const int64_t n_seg = (int64_t(P->H) + rows - 1) / rows;
  P->n_seg = int32_t(std::min<int64_t>(std::max<int64_t>(n_seg, 1), P->units));
  const int64_t waves = int64_t(P->n_win) * P->n_seg;
  if (waves > (int64_t(1) << 30)) return DWTFRAG_ERANGE;
  P->n_waves = int32_t(waves);
  P->block = block_waves(P->n_waves, cus);
  const bool last = (s == g.stages - 1);
  P->use_aes = last ? 1 : 0;
  P->key = key;
  *L_out = L;
  *C1_out = C1;
  return DWTFRAG_OK;
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}  // namespace

// Plan of a buffer whose levels fit one fused stage (levels <= kMaxFused).
int plan_single_stage(uint64_t n, uint32_t width, uint32_t levels, bool forward,
                      const dwtfrag_launch *launch, const AesKey &key, StageParams *P, int *L,
                      int *C1, uint64_t *priv_bytes) {
  if (levels > uint32_t(kMaxFused)) return DWTFRAG_EINVAL;
  Geometry g;
  const int rc = make_geometry(n, width, levels, &g);
  if (rc != DWTFRAG_OK) return rc;
  *priv_bytes = g.priv_bytes;
  return plan_stage(g, 0, forward, launch, key, P, L, C1, false);
}
// Forward stages of a planned geometry: validation of the buffers, key
// expansion, launch planning and the launches (workspace: g.ws_bytes bytes, or
// null when that is 0).
int protect_planned(const Geometry &g, const uint8_t *in, const uint8_t key[16],
                    const uint8_t nonce[16], uint8_t *priv, int16_t *pub, void *workspace,
                    const dwtfrag_launch *launch, void *stream) {
  if (!pub && g.pub_bytes) return DWTFRAG_EINVAL;  // pub may be NULL only when empty
  if (!aligned16(in) || !aligned16(priv) || !aligned16(pub) || (workspace && !aligned16(workspace)))
    return DWTFRAG_EINVAL;
  AesKey k;
  expand_key(key, nonce, &k);
  StageParams plans[kMaxStages];
  int Ls[kMaxStages], C1s[kMaxStages];
  for (int s = 0; s < g.stages; ++s) {
    const int rc = plan_stage(g, s, true, launch, k, &plans[s], &Ls[s], &C1s[s], true);
    if (rc != DWTFRAG_OK) return rc;
  }
  hipStream_t st = static_cast<hipStream_t>(stream);
  for (int s = 0; s < g.stages; ++s) {
    const bool last = (s == g.stages - 1);
    const void *src = (s == 0) ? static_cast<const void *>(in)
                               : static_cast<const char *>(workspace) + g.ws_off[s - 1];
    int16_t *dst = last ? reinterpret_cast<int16_t *>(priv)
                        : reinterpret_cast<int16_t *>(static_cast<char *>(workspace) + g.ws_off[s]);
    if (launch_fwd(Ls[s], C1s[s], s == 0, src, pub, dst, plans[s], st) != hipSuccess)
      return DWTFRAG_EDEVICE;
  }
  return DWTFRAG_OK;
}

// Static workspace of dwtfrag_protect_noalloc: one array per device, kept
// until the process ends.  Its host-side name is not a device address; the
// device address is looked up once per device (with that device current) and
// only that address is handed to kernels.  Every call on a device shares the
// array: each stage writes every element of its LL output before the next
// stage reads it, so nothing needs clearing, and calls that overlap on one
// device race on it.
static __device__ __align__(256) uint8_t scratch[kScratchBytes];

int device_scratch(void **out) {
  constexpr int kDev = 64;
  static std::mutex mu;
  static void *ptr[kDev] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kDev) return DWTFRAG_EDEVICE;
  std::lock_guard<std::mutex> lock(mu);
  if (!ptr[dev]) {
    void *p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return DWTFRAG_EDEVICE;
    ptr[dev] = p;
  }
  *out = ptr[dev];
  return DWTFRAG_OK;
}

}  // namespace dwtfrag

using namespace dwtfrag;

extern "C" {

int dwtfrag_geometry(uint64_t n, uint32_t width, uint32_t levels, dwtfrag_geom *out) {
  if (!out) return DWTFRAG_EINVAL;
  Geometry g;
  const int rc = make_geometry(n, width, levels, &g);
  if (rc != DWTFRAG_OK) return rc;
  out->n = n;
  out->width = width;
  out->height = g.H;
  out->levels = levels;
  out->ll_h = uint32_t(g.h[levels]);
  out->ll_w = uint32_t(g.w[levels]);
  out->priv_bytes = g.priv_bytes;
  out->pub_bytes = g.pub_bytes;
  out->workspace_bytes = g.ws_bytes;
  return DWTFRAG_OK;
}

uint32_t dwtfrag_default_width(uint64_t n) {
  if (n == 0) return 0;
  uint64_t r = 1;
  while (r * r < n) r <<= 1;  // smallest power of two whose square reaches n
  // r is now the smallest power of two >= sqrt(n); that equals the smallest
  // power of two >= ceil(sqrt(n)).
  return uint32_t(std::min<uint64_t>(4096, r));
}

int dwtfrag_protect(const uint8_t *in, uint64_t n, uint32_t width, uint32_t levels,
                    const uint8_t key[16], const uint8_t nonce[16], uint8_t *priv, int16_t *pub,
                    void *workspace, uint64_t workspace_bytes, const dwtfrag_launch *launch,
                    void *stream) {
  if (!in || !key || !nonce || !priv) return DWTFRAG_EINVAL;
  Geometry g;
  int rc = make_geometry(n, width, levels, &g);
  if (rc != DWTFRAG_OK) return rc;
  if (!pub && g.pub_bytes) return DWTFRAG_EINVAL;  // pub may be NULL only when empty
  if (g.ws_bytes && (!workspace || workspace_bytes < g.ws_bytes)) return DWTFRAG_EWORKSPACE;
  return protect_planned(g, in, key, nonce, priv, pub, workspace, launch, stream);
}

int dwtfrag_protect_noalloc(const uint8_t *in, uint64_t n, uint32_t width, uint32_t levels,
                            const uint8_t key[16], const uint8_t nonce[16], uint8_t *priv,
                            int16_t *pub, const dwtfrag_launch *launch, void *stream) {
  if (!in || !key || !nonce || !priv) return DWTFRAG_EINVAL;
  Geometry g;
  int rc = make_geometry(n, width, levels, &g);
  if (rc != DWTFRAG_OK) return rc;
  if (g.ws_bytes > kScratchBytes) return DWTFRAG_ESCRATCH;
  void *ws = nullptr;
  if (g.ws_bytes) {
    rc = device_scratch(&ws);
    if (rc != DWTFRAG_OK) return rc;
  }
  return protect_planned(g, in, key, nonce, priv, pub, ws, launch, stream);
}

int dwtfrag_restore(const uint8_t *priv, const int16_t *pub, uint64_t n, uint32_t width,
                    uint32_t levels, const uint8_t key[16], const uint8_t nonce[16], uint8_t *out,
                    void *workspace, uint64_t workspace_bytes, const dwtfrag_launch *launch,
                    void *stream) {
  if (!priv || !key || !nonce || !out) return DWTFRAG_EINVAL;
  Geometry g;
  int rc = make_geometry(n, width, levels, &g);
  if (rc != DWTFRAG_OK) return rc;
  if (!pub && g.pub_bytes) return DWTFRAG_EINVAL;  // pub may be NULL only when empty
  if (g.ws_bytes && (!workspace || workspace_bytes < g.ws_bytes)) return DWTFRAG_EWORKSPACE;
  if (!aligned16(out) || !aligned16(priv) || !aligned16(pub) || (workspace && !aligned16(workspace)))
    return DWTFRAG_EINVAL;
  AesKey k;
  expand_key(key, nonce, &k);
  StageParams plans[kMaxStages];
  int Ls[kMaxStages], C1s[kMaxStages];
  for (int s = 0; s < g.stages; ++s) {
    rc = plan_stage(g, s, false, launch, k, &plans[s], &Ls[s], &C1s[s], true);
    if (rc != DWTFRAG_OK) return rc;
  }
  hipStream_t st = static_cast<hipStream_t>(stream);
  for (int s = g.stages - 1; s >= 0; --s) {
    const bool last = (s == g.stages - 1);
    const int16_t *src = last ? reinterpret_cast<const int16_t *>(priv)
                              : reinterpret_cast<const int16_t *>(
                                    static_cast<const char *>(workspace) + g.ws_off[s]);
    void *dst = (s == 0) ? static_cast<void *>(out)
                         : static_cast<void *>(static_cast<char *>(workspace) + g.ws_off[s - 1]);
    if (launch_inv(Ls[s], C1s[s], s == 0, src, pub, dst, plans[s], st) != hipSuccess)
      return DWTFRAG_EDEVICE;
  }
  return DWTFRAG_OK;
}

int dwtfrag_aes128_ctr(const uint8_t *in, uint8_t *out, uint64_t nbytes, const uint8_t key[16],
                       const uint8_t nonce[16], uint64_t first_block, void *stream) {
  if (!in || !out || !key || !nonce || nbytes == 0) return DWTFRAG_EINVAL;
  AesKey k;
  expand_key(key, nonce, &k);
  if (launch_ctr(in, out, nbytes, k, first_block, static_cast<hipStream_t>(stream)) != hipSuccess)
    return DWTFRAG_EDEVICE;
  return DWTFRAG_OK;
}

int dwtfrag_autotune(const uint8_t *in, uint64_t n, uint32_t width, uint32_t levels,
                     void *scratch, uint64_t scratch_bytes, uint32_t trials,
                     dwtfrag_launch *best, float *best_us, void *stream) {
  if (!in || !scratch || !best || trials == 0) return DWTFRAG_EINVAL;
  Geometry g;
  int rc = make_geometry(n, width, levels, &g);
  if (rc != DWTFRAG_OK) return rc;
  const uint64_t o_pub = align256(g.priv_bytes);
  const uint64_t o_out = o_pub + align256(g.pub_bytes);
  const uint64_t o_ws = o_out + align256(n);
  if (scratch_bytes < o_ws + g.ws_bytes || (reinterpret_cast<uintptr_t>(scratch) & 255))
    return DWTFRAG_EWORKSPACE;
  char *base = static_cast<char *>(scratch);
  uint8_t *priv = reinterpret_cast<uint8_t *>(base);
  int16_t *pub = g.pub_bytes ? reinterpret_cast<int16_t *>(base + o_pub) : nullptr;
  uint8_t *out = reinterpret_cast<uint8_t *>(base + o_out);
  void *ws = g.ws_bytes ? base + o_ws : nullptr;
  const uint8_t key[16] = {0}, nonce[16] = {0};
  hipStream_t st = static_cast<hipStream_t>(stream);
  hipEvent_t e0, e1;
  if (hipEventCreate(&e0) != hipSuccess) return DWTFRAG_EDEVICE;
  if (hipEventCreate(&e1) != hipSuccess) {
    (void)hipEventDestroy(e0);
    return DWTFRAG_EDEVICE;
  }
  float best_t = -1.0f;
  dwtfrag_launch best_l{0, 0};
  // The default, and the heights that the kernels have: multiples of the first
  // stage's unit, up to the rows whose keystream a wavefront keeps, and no more
  // than one past the view's.  (Columns 0: the default of a stage whose
  // directions differ; elsewhere it is one of the others.)
  const int L0 = int(std::min<uint32_t>(kMaxFused, levels));
  const uint32_t rows[] = {0, 8, 16, 24, 32, 48, 64, 96, 128};
  const uint32_t cols[] = {0, 8, 16};
  const uint64_t cells = g.h[0] * g.w[0];
  rc = DWTFRAG_OK;
  for (uint32_t c : cols) {
    if (c == 0 && wide_stage(true, L0, cells) == wide_stage(false, L0, cells)) continue;
    if (levels % kMaxFused == 0 && c == 8) continue;  // a four-level stage needs 16 columns
    uint64_t tallest = 0;
    for (uint32_t r : rows) {
      if (r && (c == 0 || r % (1u << L0) || int(r) > fwd_max_rows(L0, L0 == 4 ? 16 : int(c)) || tallest >= g.h[0]))
        continue;
      tallest = r;
      const dwtfrag_launch ln{r, c};
      // one untimed pair, then `trials` timed pairs; the first failing call's
      // code is returned
      auto pair = [&]() {
        const int r = dwtfrag_protect(in, n, width, levels, key, nonce, priv, pub, ws, g.ws_bytes, &ln, st);
        return r != DWTFRAG_OK ? r
                               : dwtfrag_restore(priv, pub, n, width, levels, key, nonce, out, ws,
                                                 g.ws_bytes, &ln, st);
      };
      rc = pair();
      if (rc != DWTFRAG_OK) break;
      if (hipEventRecord(e0, st) != hipSuccess) {
        rc = DWTFRAG_EDEVICE;
        break;
      }
      for (uint32_t t = 0; t < trials && rc == DWTFRAG_OK; ++t) rc = pair();
      if (rc != DWTFRAG_OK) break;
      float ms = 0.0f;
      if (hipEventRecord(e1, st) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
          hipEventElapsedTime(&ms, e0, e1) != hipSuccess) {
        rc = DWTFRAG_EDEVICE;
        break;
      }
      const float us = 1000.0f * ms / float(trials);
      if (best_t < 0.0f || us < best_t) {
        best_t = us;
        best_l = ln;
      }
    }
    if (rc != DWTFRAG_OK) break;
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (rc != DWTFRAG_OK) return rc;
  *best = best_l;
  if (best_us) *best_us = best_t;
  return DWTFRAG_OK;
}

const char *dwtfrag_strerror(int code) {
  switch (code) {
    case DWTFRAG_OK: return "ok";
    case DWTFRAG_EINVAL: return "invalid argument (null or misaligned pointer, zero size, bad levels or launch shape)";
    case DWTFRAG_ERANGE: return "geometry out of range";
    case DWTFRAG_EDEVICE: return "HIP runtime or launch error";
    case DWTFRAG_EWORKSPACE: return "workspace missing or too small";
    case DWTFRAG_ESCRATCH: return "the transform needs more workspace than the library's 16 MiB static buffer holds";
    default: return "unknown status";
  }
}

}  // extern "C"
