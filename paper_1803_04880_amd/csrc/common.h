// Shared definitions of the HIP path: launch parameters, wavefront neighbour
// taps, and AES-128 (tables derived at compile time from GF(2^8) arithmetic).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dwtfrag {

// Levels fused into one streaming kernel; deeper transforms run as further
// stages over the LL band of the previous stage.
constexpr int kMaxFused = 4;
constexpr int kWavesPerBlock = 4;
constexpr int kBlockThreads = 64 * kWavesPerBlock;

// ----------------------------------------------------------------- AES-128 --
// FIPS-197 S-box: multiplicative inverse in GF(2^8) mod x^8+x^4+x^3+x+1, then
// the affine map b_i ^ b_{i+4} ^ b_{i+5} ^ b_{i+6} ^ b_{i+7} ^ 0x63_i.
constexpr uint8_t gf_mul(uint8_t a, uint8_t b) {
  uint8_t r = 0;
  for (int i = 0; i < 8; ++i) {
    if (b & 1) r ^= a;
    bool hi = a & 0x80;
    a = uint8_t(a << 1);
    if (hi) a ^= 0x1B;
    b >>= 1;
  }
  return r;
}

constexpr uint8_t gf_inv(uint8_t a) {
  if (a == 0) return 0;
  uint8_t r = 1, base = a;
  int e = 254;
  while (e) {
    if (e & 1) r = gf_mul(r, base);
    base = gf_mul(base, base);
    e >>= 1;
  }
  return r;
}

constexpr uint8_t rotl8(uint8_t v, int s) { return uint8_t((v << s) | (v >> (8 - s))); }

constexpr uint8_t sbox_entry(uint8_t a) {
  uint8_t b = gf_inv(a);
  return uint8_t(b ^ rotl8(b, 1) ^ rotl8(b, 2) ^ rotl8(b, 3) ^ rotl8(b, 4) ^ 0x63);
}

struct AesTables {
  uint8_t sbox[256];
  // te0[x]: MixColumns column of a substituted byte in row 0, as a
  // little-endian word (bytes 2S, S, S, 3S); rows 1..3 are byte rotations.
  uint32_t te0[256];
};

constexpr AesTables make_aes_tables() {
  AesTables t{};
  for (int x = 0; x < 256; ++x) {
    uint8_t s = sbox_entry(uint8_t(x));
    uint8_t s2 = gf_mul(s, 2), s3 = uint8_t(s2 ^ s);
    t.sbox[x] = s;
    t.te0[x] = uint32_t(s2) | (uint32_t(s) << 8) | (uint32_t(s) << 16) | (uint32_t(s3) << 24);
  }
  return t;
}

// Round keys as little-endian column words (44 words); nonce as two 64-bit
// big-endian halves.
struct AesKey {
  uint32_t rk[44];
  uint64_t nonce_hi, nonce_lo;
};

void expand_key(const uint8_t key[16], const uint8_t nonce[16], AesKey *out);

__device__ __forceinline__ uint32_t bswap32(uint32_t v) { return __builtin_bswap32(v); }

// Key material as staged in LDS: 44 round-key words, then the nonce as
// (hi low word, hi high word, lo low word, lo high word).
constexpr int kKeyWords = 48;

// Block j of the counter sequence as 4 little-endian state words.
__device__ __forceinline__ void counter_block(const uint32_t *kw, uint64_t j, uint32_t w[4]) {
  const uint64_t nhi = uint64_t(kw[44]) | (uint64_t(kw[45]) << 32);
  const uint64_t nlo = uint64_t(kw[46]) | (uint64_t(kw[47]) << 32);
  uint64_t lo = nlo + j;
  uint64_t hi = nhi + (lo < nlo ? 1ull : 0ull);
  w[0] = bswap32(uint32_t(hi >> 32));
  w[1] = bswap32(uint32_t(hi));
  w[2] = bswap32(uint32_t(lo >> 32));
  w[3] = bswap32(uint32_t(lo));
}

// One AES-128 encryption; `te` points at four 256-word tables in LDS
// (te[256 r + x] = rotl(te0[x], 8 r)), `rk` at the 44 round-key words.
// Each column of a middle round is four table words and a round-key word
// XORed together: two 3-input bit operations (truth table 0x96 = a ^ b ^ c).
// The last round takes the S-box byte (byte 1 of te0[x]) of four lookups
// with two byte permutes and joins them with the round key in one 3-input
// operation (truth table 0x56 = (a | b) ^ c).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ void aes_encrypt(const uint32_t *te, const uint32_t *rk, uint32_t w[4]) {
  uint32_t s0 = w[0] ^ rk[0], s1 = w[1] ^ rk[1], s2 = w[2] ^ rk[2], s3 = w[3] ^ rk[3];
#define DWTFRAG_TE(r, v) te[256 * (r) + (((v) >> (8 * (r))) & 0xFF)]
#pragma unroll
  for (int rnd = 1; rnd < 10; ++rnd) {
    const uint32_t t0 = xor3(xor3(DWTFRAG_TE(0, s0), DWTFRAG_TE(1, s1), DWTFRAG_TE(2, s2)), DWTFRAG_TE(3, s3), rk[4 * rnd + 0]);
    const uint32_t t1 = xor3(xor3(DWTFRAG_TE(0, s1), DWTFRAG_TE(1, s2), DWTFRAG_TE(2, s3)), DWTFRAG_TE(3, s0), rk[4 * rnd + 1]);
    const uint32_t t2 = xor3(xor3(DWTFRAG_TE(0, s2), DWTFRAG_TE(1, s3), DWTFRAG_TE(2, s0)), DWTFRAG_TE(3, s1), rk[4 * rnd + 2]);
    const uint32_t t3 = xor3(xor3(DWTFRAG_TE(0, s3), DWTFRAG_TE(1, s0), DWTFRAG_TE(2, s1)), DWTFRAG_TE(3, s2), rk[4 * rnd + 3]);
    s0 = t0; s1 = t1; s2 = t2; s3 = t3;
  }
#undef DWTFRAG_TE
  // last round: SubBytes + ShiftRows + the last round key
#define DWTFRAG_L(v, r) te[((v) >> (8 * (r))) & 0xFF]
#define DWTFRAG_LAST(a, b, c, d, k)                                                             \
  __builtin_amdgcn_bitop3_b32(__builtin_amdgcn_perm(DWTFRAG_L(b, 1), DWTFRAG_L(a, 0), 0x0c0c0501u), \
                              __builtin_amdgcn_perm(DWTFRAG_L(d, 3), DWTFRAG_L(c, 2), 0x05010c0cu), \
                              (k), 0x56)
  w[0] = DWTFRAG_LAST(s0, s1, s2, s3, rk[40]);
  w[1] = DWTFRAG_LAST(s1, s2, s3, s0, rk[41]);
  w[2] = DWTFRAG_LAST(s2, s3, s0, s1, rk[42]);
  w[3] = DWTFRAG_LAST(s3, s0, s1, s2, rk[43]);
#undef DWTFRAG_LAST
#undef DWTFRAG_L
}

static __constant__ AesTables c_aes = make_aes_tables();

// The four byte-rotated T-tables (1024 words) into LDS, loaded by the whole
// block; the caller synchronises the block afterwards.
__device__ __forceinline__ void load_aes_te(uint32_t *te) {
  for (int i = threadIdx.x; i < 256; i += blockDim.x) {
    const uint32_t v = c_aes.te0[i];
#pragma unroll
    for (int r = 0; r < 4; ++r) te[256 * r + i] = __builtin_amdgcn_alignbit(v, v, (32 - 8 * r) & 31);
  }
}

// Word i (< kKeyWords) of the LDS key block: 44 round-key words, then the
// nonce's two 64-bit halves as low / high words.
template <class K> __device__ __forceinline__ uint32_t key_word(K &key, int i) {
  if (i < 44) return key.rk[i];
  if (i == 44) return uint32_t(key.nonce_hi);
  if (i == 45) return uint32_t(key.nonce_hi >> 32);
  if (i == 46) return uint32_t(key.nonce_lo);
  return uint32_t(key.nonce_lo >> 32);
}

// Tables and key words of a block of 64 or 256 threads that uses one key, in
// two steps: the loads, and the writes to LDS once they have arrived (the
// block then synchronises).  Loads issued in between are not waited for.
struct AesLoad {
  uint32_t t[4], k;
  __device__ __forceinline__ void issue(const AesKey &key) {
    const int i = int(threadIdx.x);
    t[0] = c_aes.te0[i];
    if (blockDim.x == 64) {
#pragma unroll
      for (int j = 1; j < 4; ++j) t[j] = c_aes.te0[64 * j + i];
    }
    k = i < kKeyWords ? key_word(key, i) : 0;
  }
  __device__ __forceinline__ void finish(uint32_t *te, uint32_t *kw) const {
    const int i = int(threadIdx.x);
    put(te + i, t[0]);
    if (blockDim.x == 64) {
#pragma unroll
      for (int j = 1; j < 4; ++j) put(te + 64 * j + i, t[j]);
    }
    if (i < kKeyWords) kw[i] = k;
  }
  __device__ __forceinline__ static void put(uint32_t *te, uint32_t v) {
#pragma unroll
    for (int r = 0; r < 4; ++r) te[256 * r] = __builtin_amdgcn_alignbit(v, v, (32 - 8 * r) & 31);
  }
};

// Tables and key words together, for a block that uses one key.
template <class K> __device__ __forceinline__ void load_aes_tables(uint32_t *te, uint32_t *kw, K &key) {
  load_aes_te(te);
  for (int i = threadIdx.x; i < kKeyWords; i += blockDim.x) kw[i] = key_word(key, i);
}

// --------------------------------------------------------- launch geometry --
// One stage = up to kMaxFused levels over an H x W input.  Wavefronts own
// rectangles of the level-0 grid: window k owns columns [k*own_w, ...);
// the rows are cut into `units` units of unit_rows = 2^L rows, and segment s
// owns units [floor(s*units/n_seg), floor((s+1)*units/n_seg)), so segment
// lengths differ by at most one unit.
struct StageParams {
  int64_t n_valid;            // valid input elements (byte view: n; else H*W)
  int32_t H, W;               // stage input dims
  int32_t hdim[kMaxFused + 1], wdim[kMaxFused + 1];  // level dims, [0] = input
  int64_t off_hl[kMaxFused + 1], off_lh[kMaxFused + 1], off_hh[kMaxFused + 1];
  int32_t own_w, n_win;       // owned columns per window, number of windows
  int32_t unit_rows, units;   // 2^L, ceil(H / 2^L)
  int32_t n_seg;              // number of row segments
  int32_t halo_l;             // columns before the owned range (multiple of lane_cols)
  int32_t block;              // wavefronts per workgroup of a launch of its own
  int32_t halo_b;             // rows streamed after the owned range (before it: the
                              // forward twice as many, the inverse as many)
  int32_t n_waves;
  int32_t use_aes;            // LL output / input goes through AES-CTR
  AesKey key;
};

// Rows and columns of a view.  The launch planning and the kernels index rows
// and columns in int32 with margins of up to a window (1024 columns) and a
// unit plus halos (under 64 rows) past the end, so the limit keeps 2^16 below
// 2^31.
constexpr int32_t kMaxDim = 0x7FFF0000;

// Forward kernel: the rows of a segment are limited by the keystream that a
// wavefront holds in LDS: 16 LL rows (8 at four levels, and at one level of
// 16 columns a lane), under 9 KiB, so that four workgroups fit a compute
// unit.  A row takes its elements' blocks and two cut ones.
constexpr int fwd_ll_rows(int L, int C1) { return L == 4 || (L == 1 && C1 == 16) ? 8 : 16; }
constexpr int fwd_max_rows(int L, int C1) { return fwd_ll_rows(L, C1) << L; }
constexpr int fwd_ks_words(int L, int C1) {
  return fwd_ll_rows(L, C1) * (64 * C1 / (8 << L) + 2) * 4;
}
// Inverse kernel: the same limit; its keystream takes the window's lanes, one
// row above and one below the segment's, and a block that lanes past the
// row's end may read.
constexpr int inv_max_rows(int L, int C1) { return fwd_max_rows(L, C1); }
constexpr int inv_ks_words(int L, int C1) {
  return ((fwd_ll_rows(L, C1) + 2) * (64 * C1 / (8 << L) + 2) + 1) * 4;
}
// Wavefronts per workgroup of a launch: one where the whole grid is no more
// than two wavefronts per compute unit (each then has an LDS of its own for
// the AES lookups), else four.
constexpr int block_waves(int n_waves, int cus) { return n_waves <= 2 * cus ? 1 : kWavesPerBlock; }

// Compute units of the current device (a partition has fewer than the 256 that
// the constants of the launch rules were measured on: they go with it).
int device_cus();

// Most wavefronts of a launch: HIP takes fewer than 2^32 work-items per grid
// dimension (with the last workgroup's idle wavefronts counted).  Segments of
// the tallest kind at 8 columns a lane keep every height below it.
constexpr int32_t kMaxLaunchWaves = (1 << 26) - kWavesPerBlock;
static_assert(kMaxDim / fwd_max_rows(1, 8) < kMaxLaunchWaves, "the tallest view in one launch");

// A stage's parameters as the kernels take them (SP below): a kernel argument,
// or an entry of a batch's item table, read through the constant address
// space so that it comes by scalar loads.
using ConstStage = const __attribute__((address_space(4))) StageParams;

// Reads of a lane's `span` samples at the end of a view of n_valid elements.
// last_read_col: the last column (negative: before the row) of the row at
// element `at` from which they may be read, kMaxDim where that lies further on
// than any row is wide.  A lane past that column reads from there, and
// read_shift is by how many samples it then moves them down.
__host__ __device__ constexpr int last_read_col(int64_t n_valid, int64_t at, int span) {
  const int64_t left = n_valid - at;
  return int(left < kMaxDim + span ? left : kMaxDim + span) - span;
}
__host__ __device__ constexpr int read_shift(int c0, int last, int span) {
  const int past = c0 - last > 0 ? c0 - last : 0;
  return past < span ? past : span;
}

// Whether a view goes to the kernels of few rows, which loop over the rows
// there are, where the streaming kernel takes two whole units of 2^L rows: up
// to half a unit, and up to a whole one where the stream's last window or
// segment is of the slower kind (lanes cut by the row's end; forward, a partial
// last row).  One LL row in any case.  Measured, us forward / inverse, few rows
// against the stream: four levels of width 4096, 1 row 8 / 8 against 17 / 34,
// 8 rows 12 / 12 against 17 / 35 (16 rows: the stream 17 / 15); of width 4099,
// 1 row 8 / 10 against 37 / 35, 16 rows 18 / 27 against 37 / 36; three levels
// of width 4099, 8 rows 9 / 13 against 14 / 16; 12 rows of 1 MiB less a third,
// four levels, 20 / 35 against 27 / 26.
inline bool few_rows(const StageParams &P, int L, int C1, bool forward) {
  const bool slow = P.W % C1 != 0 || (forward && P.n_valid < int64_t(P.H) * P.W);
  return P.hdim[slow ? L : L - 1] == 1;
}

// LDS of a wavefront of the inverse of few rows: words per lane of level l's
// rows (LL, HL, LH and HH), and bytes in all.
__host__ __device__ constexpr int inv_few_words(int C1, int l, int rows) {
  return 4 * ((C1 >> (l - 1)) >= 4 ? (C1 >> (l - 1)) / 4 : 1) * rows;
}
inline unsigned inv_few_lds(const StageParams &P, int L, int C1) {
  unsigned words = 0;
  for (int l = 1; l <= L; ++l) words += inv_few_words(C1, l, P.hdim[l]);
  return 64 * 4 * words;
}

// First level-0 row of segment s (s == n_seg gives units * unit_rows).
template <class SP> __device__ __forceinline__ int seg_start(SP &P, int s) {
  return P.unit_rows * int((int64_t(s) * P.units) / P.n_seg);
}

// ------------------------------------------------------ global pointers --
// Buffer accesses go through these: a pointer into device global memory, so
// that loads and stores compile to global (not flat) instructions also where
// the address was read from memory (batch items), which the compiler cannot
// place in an address space by itself.  Cast with glob() first, then change
// the pointee type.
template <class T> using gptr = __attribute__((address_space(1))) T *;
template <class T> __device__ __forceinline__ gptr<T> glob(T *p) { return (gptr<T>)p; }
// 8- and 16-byte vectors for those accesses (plain vector types, which can be
// read from any address space).
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// n dwords as one vector.
template <int n> using Vec = uint32_t __attribute__((ext_vector_type(n)));
// The same at any byte address: rows of a width that is no multiple of the
// vector are read unaligned.
typedef u32x2 u32x2_u __attribute__((aligned(1)));
typedef u32x4 u32x4_u __attribute__((aligned(1)));

// A pointer that is the same in every lane, in scalar registers.
template <class T> __device__ __forceinline__ T *uniform_ptr(T *p) {
  const uint64_t a = reinterpret_cast<uint64_t>(p);
  return reinterpret_cast<T *>(uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(int(a)))) |
                               (uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(int(a >> 32)))) << 32));
}

// ------------------------------------------------------- wavefront taps --
// wave_shl:1 -> lane i receives lane i+1; wave_shr:1 -> lane i receives
// lane i-1 (the lane with no source receives 0, or `none`).
__device__ __forceinline__ int from_next_lane(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x130, 0xF, 0xF, false);
}
__device__ __forceinline__ int from_prev_lane(int v, int none = 0) {
  return __builtin_amdgcn_update_dpp(none, v, 0x138, 0xF, 0xF, false);
}

__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace dwtfrag
