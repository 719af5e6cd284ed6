// Inverse path: AES-CTR decryption of the LL band fused with the multi-level
// inverse 5/3 lifting, as one streaming kernel (Ch. 5 section 5.2.3: the map
// is an invertible integer-to-integer map, so restore is exact).
//
// Within a level the vertical pass is undone first, then the horizontal one
// (the reverse of the forward order).  Step k of level l takes LL_l row k and
// the detail rows k of HL_l / LH_l / HH_l and yields rows 2k-1 and 2k of the
// level-(l-1) grid, which are inverted horizontally and are LL rows of the
// next finer level; level 1 yields output rows.
//
// One wavefront owns a rectangle of the output (a column window times a short
// row segment).  Its unit u is step u of the last level with the steps that
// follow from it, rows 2^L (u-1) + 1 .. 2^L u, as straight-line code: each
// step's detail rows are loaded a few steps ahead into a ring of registers,
// rows go out through buffer stores without branches (rows and lanes that are
// not owned are dropped by the hardware's range check), so that the waits for
// loads count past the stores in flight.  The keystream of the LL rows is
// computed into LDS while the first rows are on their way.
//
// What bounds it is HBM at large sizes; at an image's size each SIMD has one
// or two wavefronts, and it is their latency.  Measured against a wavefront
// per long segment with LDS queues between the levels and a launch of its own
// for the exact redo: 256 MiB at three levels 200 -> 162 us (5.0 TB/s), 16
// MiB 35.2 -> 17.4 us, 12 MB of width 3001 at two levels 36 -> 24 us, 64 MiB
// at six levels, both ways, 173 -> 133 us.
#pragma once

#include "lift.h"
#include "pack.h"

namespace dwtfrag {

// A wavefront's rectangle and window.
struct InvRect {
  int X0, X1, Y0, Y1;   // owned rectangle (level 0), X1 / Y1 exclusive
  int cbase;            // first column of the window
  bool last_win, last_seg;

  template <class SP> __device__ __forceinline__ InvRect(SP &G, int wave) {
    const int win = wave % G.n_win, seg = wave / G.n_win;
    last_win = (win == G.n_win - 1);
    last_seg = (seg == G.n_seg - 1);
    X0 = win * G.own_w;
    X1 = last_win ? G.W : X0 + G.own_w;
    Y0 = seg_start(G, seg);
    Y1 = last_seg ? G.H : seg_start(G, seg + 1);
    cbase = (win == 0) ? 0 : X0 - G.halo_l;
  }
};

// Keystream of LL rows [k0, k1) for the window's lanes: row r's blocks start
// at block r * nb; lane columns outside the band have none.
template <int L, int C1> struct InvKeys {
  const uint32_t *ks;
  int k0, nb, cl0, cl1;   // first row, blocks per row, the window's LL columns [cl0, cl1)

  template <class SP>
  __device__ __forceinline__ InvKeys(SP &G, const InvRect &B, const uint32_t *lds, int first)
      : ks(lds), k0(first) {
    cl0 = min(G.wdim[L], B.cbase >> L);
    cl1 = min(G.wdim[L], (B.cbase + 64 * C1) >> L);
    nb = (2 * (cl1 - cl0) + 30) >> 4;
  }
  template <class SP>
  __device__ __forceinline__ void fill(SP &G, uint32_t *lds, int k1, const uint32_t *te,
                                       const uint32_t *kw, int lane) const {
    const int total = (k1 - k0) * nb;
    const int step_r = 64 / nb, step_c = 64 % nb;
    int r = lane / nb, c = lane % nb;
#pragma unroll 1
    for (int i = lane; i < total; i += 64) {
      const int64_t e = int64_t(k0 + r) * G.wdim[L] + cl0;  // the row's first element
      const int64_t b = (e >> 3) + c;
      if (8 * b < e + (cl1 - cl0)) {
        uint32_t w[4];
        counter_block(kw, uint64_t(b), w);
        aes_encrypt(te, kw, w);
        *reinterpret_cast<uint4 *>(lds + 4 * i) = make_uint4(w[0], w[1], w[2], w[3]);
      }
      c += step_c;
      r += step_r;
      if (c >= nb) { c -= nb; ++r; }
    }
  }
  // Byte offset of LL row k's first keystream byte (at column cl0).
  template <class SP> __device__ __forceinline__ int row(SP &G, int k) const {
    return (k - k0) * 16 * nb + (2 * (k * (G.wdim[L] & 7) + cl0) & 15);
  }
};

// The stream in 32-bit arithmetic, exact for any fragment contents.  Used for
// rectangles whose fragments hold a value outside the packed stream's range
// (none that protect made).
template <int L, int C1, bool U8OUT, class SP>
struct InvWave {
  template <int l> static constexpr int C = C1 >> (l - 1);

  SP &P;
  const InvRect &B;
  const int16_t *llin;     // LL_L (priv bytes or int16 scratch)
  const int16_t *pub;
  void *out;
  const InvKeys<L, C1> &ks;
  int lane;
  int c0;

  int Dp1[C<1>], Xp1[C<1>];
  int Dp2[L >= 2 ? C<2> : 1], Xp2[L >= 2 ? C<2> : 1];
  int Dp3[L >= 3 ? C<3> : 1], Xp3[L >= 3 ? C<3> : 1];
  int Dp4[L >= 4 ? C<4> : 1], Xp4[L >= 4 ? C<4> : 1];
  int k0[kMaxFused + 1];   // first step index of each level's stream

  template <int l> __device__ auto &Dp() {
    if constexpr (l == 1) return Dp1; else if constexpr (l == 2) return Dp2;
    else if constexpr (l == 3) return Dp3; else return Dp4;
  }
  template <int l> __device__ auto &Xp() {
    if constexpr (l == 1) return Xp1; else if constexpr (l == 2) return Xp2;
    else if constexpr (l == 3) return Xp3; else return Xp4;
  }

  // U values of a band row from column bc (zeros past the row's end).
  template <int U> __device__ __forceinline__ static void load(const int16_t *row, int bc, int cols, int (&v)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = bc + u < cols ? int(glob(row)[bc + u]) : 0;
  }

  // Row i of the level-(l-1) grid after the vertical inverse of level l:
  // undo the horizontal pass, then hand it down.
  template <int l> __device__ __forceinline__ void emit_row(int (&x)[C<l>], int i) {
    hinv_any<C<l>>(x, c0 >> (l - 1), P.wdim[l - 1], true);
    if constexpr (l > 1) {
      push_ll<l - 1>(x, i);
    } else {
      if (i < B.Y0 || (!B.last_seg && i >= B.Y1)) return;
      if (c0 < B.X0 || (!B.last_win && c0 >= B.X1)) return;
      const int64_t idx = int64_t(i) * P.W + c0;
      const int64_t lim = min(int64_t(P.W - c0), P.n_valid - idx);
#pragma unroll
      for (int t = 0; t < C1; ++t)
        if (t < lim) {
          if constexpr (U8OUT) glob(static_cast<uint8_t *>(out))[idx + t] = uint8_t(x[t]);
          else glob(static_cast<int16_t *>(out))[idx + t] = int16_t(x[t]);
        }
    }
  }

  // Step k of level l: LL_l row k arrives (values of this lane's LL columns).
  // The step yields up to three rows of the level-(l-1) grid (2k-1, 2k and,
  // at the end of an even-length signal, 2k+1), emitted from one call site.
  template <int l> __device__ __forceinline__ void push_ll(const int (&ll)[C<l> / 2], int k) {
    constexpr int CC = C<l>;
    constexpr int U = CC / 2;
    const int N = P.hdim[l - 1];
    const int wl = P.wdim[l], wh = P.wdim[l - 1] - wl;
    const int bc = c0 >> l;
    int hl[U];
    load<U>(pub + P.off_hl[l] + int64_t(k) * wh, bc, wh, hl);
    int S[CC];
#pragma unroll
    for (int u = 0; u < U; ++u) { S[2 * u] = ll[u]; S[2 * u + 1] = hl[u]; }
    auto &Dv = Dp<l>();
    auto &Xv = Xp<l>();
    int R0[CC], R1[CC], R2[CC];
    int e_begin = 1, e_end = 2;
    if (N == 1) {  // no vertical pass at this level: the row is row 0
#pragma unroll
      for (int t = 0; t < CC; ++t) R1[t] = S[t];
    } else {
      int Dn[CC];
      if (2 * k + 1 < N) {
        int lh[U], hh[U];
        load<U>(pub + P.off_lh[l] + int64_t(k) * wl, bc, wl, lh);
        load<U>(pub + P.off_hh[l] + int64_t(k) * wh, bc, wh, hh);
#pragma unroll
        for (int u = 0; u < U; ++u) { Dn[2 * u] = lh[u]; Dn[2 * u + 1] = hh[u]; }
      } else {  // odd length, last step: d(N) = d(N-2)
#pragma unroll
        for (int t = 0; t < CC; ++t) Dn[t] = Dv[t];
      }
      const bool top = (k == 0);
#pragma unroll
      for (int t = 0; t < CC; ++t) {
        const int X = S[t] - (((top ? Dn[t] : Dv[t]) + Dn[t] + 2) >> 2);
        R0[t] = Dv[t] + ((Xv[t] + X) >> 1);  // x(2k-1)
        R1[t] = X;                             // x(2k)
        R2[t] = Dn[t] + X;                     // x(2k+1) when 2k+1 == N-1
        Dv[t] = Dn[t];
        Xv[t] = X;
      }
      if (k != k0[l]) e_begin = 0;
      if (2 * k + 1 == N - 1) e_end = 3;
    }
#pragma unroll 1
    for (int e = e_begin; e < e_end; ++e) {
      int row[CC];
#pragma unroll
      for (int t = 0; t < CC; ++t) row[t] = e == 0 ? R0[t] : (e == 1 ? R1[t] : R2[t]);
      emit_row<l>(row, 2 * k - 1 + e);
    }
  }

  __device__ __forceinline__ void run() {
    c0 = B.cbase + lane * C1;
    const int kbeg = ks.k0, kend = min(P.hdim[L], (B.Y1 + P.halo_b) >> L);
#pragma unroll
    for (int l = 1; l <= L; ++l) k0[l] = kbeg << (L - l);
#pragma unroll
    for (int t = 0; t < C<1>; ++t) { Dp1[t] = 0; Xp1[t] = 0; }
#pragma unroll
    for (int t = 0; t < (L >= 2 ? C<2> : 1); ++t) { Dp2[t] = 0; Xp2[t] = 0; }
#pragma unroll
    for (int t = 0; t < (L >= 3 ? C<3> : 1); ++t) { Dp3[t] = 0; Xp3[t] = 0; }
#pragma unroll
    for (int t = 0; t < (L >= 4 ? C<4> : 1); ++t) { Dp4[t] = 0; Xp4[t] = 0; }
    constexpr int U = C<L> / 2;
    const int wl = P.wdim[L], bc = c0 >> L;
#pragma unroll 1
    for (int k = kbeg; k < kend; ++k) {
      int ll[U];
      load<U>(llin + int64_t(k) * wl, bc, wl, ll);
      if (P.use_aes) {
        const uint16_t *p = reinterpret_cast<const uint16_t *>(reinterpret_cast<const char *>(ks.ks) + ks.row(P, k)) + (bc - ks.cl0);
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (bc + u < wl) ll[u] = int(int16_t(uint16_t(ll[u]) ^ p[u]));
      }
      push_ll<L>(ll, k);
    }
  }
};

// A lane's M int16 of a band row, as loaded: packed words, or one value kept
// in its 16 bits (widened at the load, it would have to be waited for there).
template <int M> struct RowWords {
  Vec<M / 2> v;
  __device__ __forceinline__ uint32_t operator[](int j) const { return v[j]; }
  __device__ __forceinline__ static RowWords load(gptr<const char> p) {
    typedef Vec<M / 2> Unaligned __attribute__((aligned(1)));
    return {*(gptr<const Unaligned>)p};
  }
};
template <> struct RowWords<1> {
  uint16_t v;
  __device__ __forceinline__ uint32_t operator[](int) const { return v; }
  __device__ __forceinline__ static RowWords load(gptr<const char> p) { return {*(gptr<const uint16_t>)p}; }
};

// Packed form of the stream (two int16 samples per register, the forward's
// layout: E = lows, O = highs, see pack.h).  Exact when every value a level
// reads (LL row, HL, LH, HH) lies in [-4096, 4095]: then the vertical
// inverse gives |x| <= 10240, the horizontal one evens <= 15360 and odds
// <= 25600, and no sum exceeds 30720, so 16 bits never wrap.  Fragments made
// by protect stay far inside that range.  The stream checks every value it
// reads; run() returns false when one was outside, and the caller then redoes
// the rectangle with the 32-bit stream (same output bytes as the exact
// integer inverse for any fragments).
//
// GEN: windows whose right end cuts a lane's columns, levels of one row, and
// without TAIL wavefronts that write the view's partial last row: per-lane
// edge masks, cut lanes stored in pieces, checked loads at the ends of the
// fragments.  All others run the plain form, where an edge of the row can only
// lie at a lane's boundary.
// TAIL: the kernels of views with a partial last row, whose plain form stores
// that row in pieces by itself (16 MiB of width 4088 at three levels 35.5 ->
// 18.7 us; in the kernels of whole views the checks would cost 3%).
template <int L, int C1, bool U8OUT, bool GEN, bool TAIL, class SP>
struct InvWavePk {
  template <int l> static constexpr int M = (C1 >> (l - 1)) / 2;  // evens per lane at level l
  template <int l> static constexpr int NP = Pk<M<l>>::P;         // words per parity
  template <int l> static constexpr int R = 2 * NP<l>;            // words per row: E then O
  template <int l> static constexpr int NS = 1 << (L - l);        // steps of level l per unit
  // steps of level l in flight: level 1 holds 4 (8 output rows), the others
  // the same time or one step
  template <int l> static constexpr int Q = (4 >> (l - 1)) > 0 ? (4 >> (l - 1)) : 1;
  static constexpr int UPL = NS<1> >= 4 ? 1 : 4 / NS<1>;          // units per loop trip
  static constexpr int U = 1 << L;
  static constexpr uint32_t kBias = 0x10001000u;   // [-4096, 4095] -> [0, 8191]
  static constexpr uint32_t kOutside = 0xE000E000u;
  static constexpr uint32_t kNoLane = 0x80000000u;
  static constexpr int kStoreAux = 2;  // nt

  SP &P;
  const InvRect &B;
  const int16_t *llin;
  const int16_t *pub;
  void *out;
  const InvKeys<L, C1> &ks;
  int lane;
  int c0;
  uint32_t chk;            // OR of every biased value read
  bool redge;              // the row ends with this lane's last column
  int vedge;               // the unit touches the last rows of a level
  uint32_t so;             // this lane's byte offset in an output row, or past its end
  char *prow;              // the next output row
  int ks_off;              // this lane's bytes in a keystream row
  int ulast;               // the segment's last unit
  const char *pHL[L + 1], *pLH[L + 1], *pHH[L + 1], *pLL;  // the rows loaded next
  int last_h[L + 1], last_d[L + 1];                        // the last rows of HL, and of LH and HH

  __device__ __forceinline__ InvWavePk(SP &P_, const InvRect &B_, const int16_t *llin_, const int16_t *pub_,
                                       void *out_, const InvKeys<L, C1> &ks_, int lane_)
      : P(P_), B(B_), llin(llin_), pub(pub_), out(out_), ks(ks_), lane(lane_) {}

  // detail rows of the next steps of each level, as loaded (band order is
  // the packed order: HL / HH words are O words, LH words E words), and the
  // next LL rows
  template <int l> using Words = RowWords<(M<l> > 0 ? M<l> : 1)>;
  Words<1> Fh1[Q<1>], Fl1[Q<1>], Fx1[Q<1>];
  Words<2> Fh2[Q<2>], Fl2[Q<2>], Fx2[Q<2>];
  Words<3> Fh3[Q<3>], Fl3[Q<3>], Fx3[Q<3>];
  Words<4> Fh4[Q<4>], Fl4[Q<4>], Fx4[Q<4>];
  Words<L> F0[Q<L>];
  // the first step's rows: details k - 1 and k, HL row k
  Words<1> Ih1, Il1[2], Ix1[2];
  Words<2> Ih2, Il2[2], Ix2[2];
  Words<3> Ih3, Il3[2], Ix3[2];
  Words<4> Ih4, Il4[2], Ix4[2];
  Words<L> I0;
  // vertical state: previous detail row and previous even row (E then O)
  uint32_t Dp1[R<1>], Xp1[R<1>];
  uint32_t Dp2[R<2>], Xp2[R<2>];
  uint32_t Dp3[R<3>], Xp3[R<3>];
  uint32_t Dp4[R<4>], Xp4[R<4>];

#define DWTFRAG_BY_LEVEL(name)                                                        \
  template <int l> __device__ __forceinline__ auto &name() {                          \
    if constexpr (l == 1) return name##1; else if constexpr (l == 2) return name##2;  \
    else if constexpr (l == 3) return name##3; else return name##4;                   \
  }
  DWTFRAG_BY_LEVEL(Fh) DWTFRAG_BY_LEVEL(Fl) DWTFRAG_BY_LEVEL(Fx)
  DWTFRAG_BY_LEVEL(Ih) DWTFRAG_BY_LEVEL(Il) DWTFRAG_BY_LEVEL(Ix)
  DWTFRAG_BY_LEVEL(Dp) DWTFRAG_BY_LEVEL(Xp)
#undef DWTFRAG_BY_LEVEL

  template <int n> __device__ __forceinline__ void check(const uint32_t (&w)[n]) {
    if constexpr (n == 1) {
      chk |= pk_add(w[0], kBias);
    } else {
#pragma unroll
      for (int j = 0; j + 1 < n; j += 2) chk = chk | pk_add(w[j], kBias) | pk_add(w[j + 1], kBias);
    }
  }

  // ---- loads -------------------------------------------------------------
  // This lane's M<l> values of the band row at `row` (cols columns; left is
  // what the fragment holds from the row's start on).  The general form reads
  // past a row's end, but not past the fragment's: lanes there read its last
  // M<l> values, and the step shifts them into place (realign).
  template <int l>
  __device__ __forceinline__ Words<l> load_row(const int16_t *row, int cols, int64_t left) const {
    constexpr int Mv = M<l>;
    const int bc = c0 >> l;
    int last = cols - Mv;
    if constexpr (GEN) {
      last = last_col<l>(left);
      row += min(last, 0);
    }
    const uint32_t at = 2u * uint32_t(min(bc, last) - (GEN ? min(last, 0) : 0));
    const gptr<const char> src = glob(reinterpret_cast<const char *>(uniform_ptr(row))) + at;
    return Words<l>::load(src);
  }
  // Last column (negative: before the row) from which M<l> values may be read.
  template <int l> __device__ __forceinline__ static int last_col(int64_t left) {
    return int(min(left - M<l>, int64_t(1) << 30));
  }
  // Values loaded from last_col instead of this lane's first column.
  template <int l> __device__ __forceinline__ void realign(uint32_t (&w)[NP<l>], int64_t left) const {
    const int sh = max((c0 >> l) - last_col<l>(left), 0);
#pragma unroll
    for (int b = 1; b < M<l>; b *= 2)
#pragma unroll
      for (int j = 0; j < NP<l>; ++j) {
        const uint32_t v = b == 1 ? (j + 1 < NP<l> ? align16(w[j + 1 < NP<l> ? j + 1 : j], w[j]) : w[j] >> 16)
                                  : (j + b / 2 < NP<l> ? w[j + b / 2 < NP<l> ? j + b / 2 : j] : 0u);
        w[j] = (sh & b) ? v : w[j];
      }
  }
  // Whether row k of a band of `rows` rows may end so close to the
  // fragment's end (each row holds one value at least).
  template <int l> __device__ __forceinline__ static bool near_end(int k, int rows) { return k + M<l> >= rows; }
  // Rows k of a level's bands, clamped to the segment's last step (what is
  // loaded ahead of it is not used, and comes from the caches) and to the rows
  // there are (a level of one row has no LH / HH rows: not used either).
  __device__ __forceinline__ int64_t pub_end() const {
    return P.off_hh[1] + int64_t(P.hdim[0] - P.hdim[1]) * (P.wdim[0] - P.wdim[1]);
  }
  template <int l> __device__ __forceinline__ int64_t at_hl(int k) const {
    return P.off_hl[l] + int64_t(min(k, min(NS<l> * ulast, P.hdim[l] - 1))) * (P.wdim[l - 1] - P.wdim[l]);
  }
  template <int l> __device__ __forceinline__ Words<l> load_hl(int k) const {
    const int64_t at = at_hl<l>(k);
    return load_row<l>(pub + at, P.wdim[l - 1] - P.wdim[l], GEN ? pub_end() - at : 0);
  }
  // The ring's loads, row k of HL, of LH and HH, of LL: from pointers that
  // move on while there is a next row (a row's address from its index is some
  // ten scalar instructions, and a lone wavefront issues those one by one: 16
  // MiB at three levels 18.3 -> 17.4 us).
  __device__ __forceinline__ static const char *advance(const char *p, bool more, int cols) {
    return uniform_ptr(p + (more ? 2u * uint32_t(cols) : 0u));
  }
  __device__ __forceinline__ int64_t left_at(const char *p) const {
    return GEN ? (reinterpret_cast<const char *>(pub + pub_end()) - p) >> 1 : 0;
  }
  template <int l> __device__ __forceinline__ void ring_start(int k) {
    const int wl = P.wdim[l], wh = P.wdim[l - 1] - wl;
    const int rows = P.hdim[l - 1] - P.hdim[l];
    last_h[l] = min(NS<l> * ulast, P.hdim[l] - 1);
    last_d[l] = min(NS<l> * ulast, rows - 1);
    const int kd = max(min(k, last_d[l]), 0);
    pHL[l] = uniform_ptr(reinterpret_cast<const char *>(pub + at_hl<l>(k)));
    pLH[l] = uniform_ptr(reinterpret_cast<const char *>(pub + P.off_lh[l] + int64_t(kd) * wl));
    pHH[l] = uniform_ptr(reinterpret_cast<const char *>(pub + P.off_hh[l] + int64_t(kd) * wh));
  }
  template <int l> __device__ __forceinline__ void next_rows(int k, Words<l> &h, Words<l> &lo, Words<l> &hi) {
    const int wl = P.wdim[l], wh = P.wdim[l - 1] - wl;
    h = load_row<l>(reinterpret_cast<const int16_t *>(pHL[l]), wh, left_at(pHL[l]));
    lo = load_row<l>(reinterpret_cast<const int16_t *>(pLH[l]), wl, left_at(pLH[l]));
    hi = load_row<l>(reinterpret_cast<const int16_t *>(pHH[l]), wh, left_at(pHH[l]));
    pHL[l] = advance(pHL[l], k < last_h[l], wh);
    pLH[l] = advance(pLH[l], k < last_d[l], wl);
    pHH[l] = advance(pHH[l], k < last_d[l], wh);
  }
  __device__ __forceinline__ Words<L> next_ll(int k) {
    const int wl = P.wdim[L];
    const Words<L> w = load_row<L>(reinterpret_cast<const int16_t *>(pLL), wl,
                                   GEN ? (reinterpret_cast<const char *>(llin + int64_t(P.hdim[L]) * wl) - pLL) >> 1 : 0);
    pLL = advance(pLL, k < last_h[L], wl);
    return w;
  }
  template <int l> __device__ __forceinline__ void load_d(int k, Words<l> &lo, Words<l> &hi) const {
    const int wl = P.wdim[l], wh = P.wdim[l - 1] - wl;
    const int rows = P.hdim[l - 1] - P.hdim[l];
    k = max(min(k, min(NS<l> * ulast, rows - 1)), 0);
    const int64_t al = P.off_lh[l] + int64_t(k) * wl, ah = P.off_hh[l] + int64_t(k) * wh;
    lo = load_row<l>(pub + al, wl, GEN ? pub_end() - al : 0);
    hi = load_row<l>(pub + ah, wh, GEN ? pub_end() - ah : 0);
  }
  // Clears what a lane that the row's end cuts holds past it, so that the
  // check sees the row's own values only.
  template <int l> __device__ __forceinline__ void inside(uint32_t (&a)[R<l>], uint32_t (&b)[R<l>]) const {
    const int wl = P.wdim[l], wh = P.wdim[l - 1] - wl;
    int nl = wl - (c0 >> l), nh = wh - (c0 >> l);
    // (made anew at each step: kept, the masks would need registers)
    asm volatile("" : "+v"(nl), "+v"(nh));
#pragma unroll
    for (int j = 0; j < NP<l>; ++j) {
      const uint32_t ml = (nl > 2 * j ? 0xFFFFu : 0u) | (nl > 2 * j + 1 ? 0xFFFF0000u : 0u);
      const uint32_t mh = (nh > 2 * j ? 0xFFFFu : 0u) | (nh > 2 * j + 1 ? 0xFFFF0000u : 0u);
      a[j] &= ml;
      b[j] &= ml;
      a[NP<l> + j] &= mh;
      b[NP<l> + j] &= mh;
    }
  }
  // The highs of x (row k of HL), and x (row k of LH and HH), as loaded.
  template <int l> __device__ __forceinline__ void realign_hl(uint32_t (&x)[R<l>], int k) const {
    if (!near_end<l>(k, P.hdim[l])) return;
    uint32_t w[NP<l>];
#pragma unroll
    for (int j = 0; j < NP<l>; ++j) w[j] = x[NP<l> + j];
    realign<l>(w, pub_end() - at_hl<l>(k));
#pragma unroll
    for (int j = 0; j < NP<l>; ++j) x[NP<l> + j] = w[j];
  }
  template <int l> __device__ __forceinline__ void realign_d(uint32_t (&x)[R<l>], int k) const {
    const int wl = P.wdim[l], wh = P.wdim[l - 1] - wl;
    const int rows = P.hdim[l - 1] - P.hdim[l];
    if (!near_end<l>(k, rows)) return;
    k = max(min(k, rows - 1), 0);
    uint32_t w[2][NP<l>];
#pragma unroll
    for (int j = 0; j < NP<l>; ++j) { w[0][j] = x[j]; w[1][j] = x[NP<l> + j]; }
    realign<l>(w[0], pub_end() - P.off_lh[l] - int64_t(k) * wl);
    realign<l>(w[1], pub_end() - P.off_hh[l] - int64_t(k) * wh);
#pragma unroll
    for (int j = 0; j < NP<l>; ++j) { x[j] = w[0][j]; x[NP<l> + j] = w[1][j]; }
  }
  __device__ __forceinline__ void realign_ll(uint32_t (&w)[NP<L>], int k) const {
    if constexpr (GEN) {
      if (!near_end<L>(k, P.hdim[L])) return;
      realign<L>(w, int64_t(P.hdim[L] - min(k, P.hdim[L] - 1)) * P.wdim[L]);
    }
  }
  __device__ __forceinline__ Words<L> load_ll(int k) const {
    const int wl = P.wdim[L];
    const int64_t at = int64_t(min(k, min(ulast, P.hdim[L] - 1))) * wl;
    return load_row<L>(llin + at, wl, GEN ? int64_t(P.hdim[L]) * wl - at : 0);
  }

  // ---- one row -----------------------------------------------------------
  // Row i of the level-(l-1) grid after the vertical inverse of level l, one
  // of step J's two.
  template <int l> __device__ __forceinline__ void lift_row(const uint32_t (&x)[R<l>], uint32_t (&E)[NP<l>],
                                                            uint32_t (&O)[NP<l>]) const {
#pragma unroll
    for (int j = 0; j < NP<l>; ++j) { E[j] = x[j]; O[j] = x[NP<l> + j]; }
    if constexpr (GEN) hinv_pk_any<M<l>>(E, O, c0 >> (l - 1), P.wdim[l - 1], true);
    else hinv_pk_lanes<M<l>>(E, O, redge);
  }
  template <int l> __device__ __forceinline__ void to_ll(const uint32_t (&x)[R<l>], uint32_t (&ll)[NP<l - 1>]) const {
    uint32_t E[NP<l>], O[NP<l>];
    lift_row<l>(x, E, O);
#pragma unroll
    for (int j = 0; j < NP<l>; ++j) {
      ll[2 * j] = lo_halves(E[j], O[j]);
      if constexpr (M<l> >= 2) ll[2 * j + 1] = hi_halves(E[j], O[j]);
    }
  }
  // Output row: keep is -1 where the row is owned, i its index.
  // LAST: it may be the view's last row.
  template <bool LAST> __device__ __forceinline__ void put_row(const uint32_t (&x)[R<1>], int i, int keep) {
    uint32_t E[NP<1>], O[NP<1>];
    lift_row<1>(x, E, O);
    constexpr int ES = U8OUT ? 1 : 2, RB = C1 * ES, RWd = RB / 4;
    uint32_t w[RWd];
    if constexpr (U8OUT) {
#pragma unroll
      for (int q = 0; q < RWd; ++q) w[q] = __builtin_amdgcn_perm(O[q], E[q], 0x06020400u);
    } else {
#pragma unroll
      for (int q = 0; q < RWd / 2; ++q) {
        w[2 * q] = lo_halves(E[q], O[q]);
        w[2 * q + 1] = hi_halves(E[q], O[q]);
      }
    }
    const bool part = LAST && (GEN || TAIL) && i == P.H - 1;
    const int cols = part ? int(P.n_valid - int64_t(P.H - 1) * P.W) : P.W;
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(
        uniform_ptr(prow), 0, __builtin_amdgcn_readfirstlane((cols * ES) & keep), 0x00027000);
    prow = uniform_ptr(prow + int64_t(P.W) * ES);
    uint32_t off = so;
    if (GEN || part) {
      // a lane that the row's end cuts stores its first nv bytes in pieces of
      // 16, 8, 4, 2 and 1, where nv has that bit
      const int nv = (cols - c0) * ES;
      const bool cut = nv > 0 && nv < RB && off != kNoLane;
      const auto at = [&](int bit) { return cut && (nv & bit) ? off + (nv & (0x1F & ~(2 * bit - 1))) : kNoLane; };
      const auto word = [&](int n) {  // word n, n below RWd
        uint32_t v = w[0];
#pragma unroll
        for (int j = 1; j < RWd; ++j) v = n == j ? w[j] : v;
        return v;
      };
      if constexpr (RB > 16)
        __builtin_amdgcn_raw_buffer_store_b128(u32x4{w[0], w[1], w[2 % RWd], w[3 % RWd]}, rsrc, at(16), 0, kStoreAux);
      if constexpr (RB > 8) {
        const int b = (nv & 16) >> 2;
        __builtin_amdgcn_raw_buffer_store_b64(u32x2{word(b), word(b + 1)}, rsrc, at(8), 0, kStoreAux);
      }
      __builtin_amdgcn_raw_buffer_store_b32(word((nv & 24) >> 2), rsrc, at(4), 0, kStoreAux);
      const uint32_t rest = word((nv & 28) >> 2);
      __builtin_amdgcn_raw_buffer_store_b16(uint16_t(rest), rsrc, at(2), 0, kStoreAux);
      if constexpr (ES == 1)
        __builtin_amdgcn_raw_buffer_store_b8(uint8_t((nv & 2) ? rest >> 16 : rest), rsrc, at(1), 0, kStoreAux);
      if (nv < RB) off = kNoLane;
    }
    if constexpr (RWd == 2) {
      __builtin_amdgcn_raw_buffer_store_b64(u32x2{w[0], w[1]}, rsrc, off, 0, kStoreAux);
    } else {
#pragma unroll
      for (int q = 0; q < RWd; q += 4)
        __builtin_amdgcn_raw_buffer_store_b128(u32x4{w[q], w[q + 1], w[q + 2], w[q + 3]}, rsrc, off + 4 * q, 0,
                                               kStoreAux);
    }
  }

  // ---- one level ---------------------------------------------------------
  // Step J of unit u at level l (step k = NS u - NS + 1 + J): ll is LL row k.
  // S: the unit's place in the loop trip, which fixes the ring slots.  CHK:
  // the unit may touch the last rows of a level or of the segment, where
  // d(N) = d(N-2) and x(N) = x(N-2).
  template <int l, int J, int S, bool CHK>
  __device__ __forceinline__ void step(int u, const uint32_t (&ll)[NP<l>]) {
    constexpr int Np = NP<l>, Rl = R<l>;
    constexpr int slot = (S * NS<l> + J) % Q<l>;
    const int k = NS<l> * u - NS<l> + 1 + J;
    const int N = P.hdim[l - 1];
    auto &Dv = Dp<l>();
    auto &Xv = Xp<l>();
    uint32_t Sv[Rl], Dn[Rl];
#pragma unroll
    for (int j = 0; j < Np; ++j) {
      Sv[j] = ll[j];
      Sv[Np + j] = Fh<l>()[slot][j];
      Dn[j] = Fl<l>()[slot][j];
      Dn[Np + j] = Fx<l>()[slot][j];
    }
    if constexpr (GEN) {
      realign_hl<l>(Sv, k);
      realign_d<l>(Dn, k);
      inside<l>(Sv, Dn);
    }
    check(Sv);
    check(Dn);
    if (CHK && vedge && 2 * k + 1 >= N) {
#pragma unroll
      for (int t = 0; t < Rl; ++t) Dn[t] = N == 1 ? 0u : Dv[t];
    }
    uint32_t X[Rl], Ra[Rl];
#pragma unroll
    for (int t = 0; t < Rl; ++t) X[t] = pk_sub(Sv[t], pk_sra(pk_add(pk_add(Dv[t], Dn[t]), 0x00020002u), 2));
    if (CHK && vedge && 2 * k >= N) {
#pragma unroll
      for (int t = 0; t < Rl; ++t) X[t] = Xv[t];
    }
#pragma unroll
    for (int t = 0; t < Rl; ++t) {
      Ra[t] = pk_add(Dv[t], pk_sra(pk_add(Xv[t], X[t]), 1));
      copy(Dv[t], Dn[t]);
      Xv[t] = X[t];
    }
    // the slot is free: the step Q ahead
    free_regs(Dv, X, chk);
    next_rows<l>(k + Q<l>, Fh<l>()[slot], Fl<l>()[slot], Fx<l>()[slot]);
    if constexpr (l > 1) {
      uint32_t la[NP<l - 1>];
      to_ll<l>(Ra, la);
      step<l - 1, 2 * J, S, CHK>(u, la);
      to_ll<l>(X, la);
      step<l - 1, 2 * J + 1, S, CHK>(u, la);
    } else {
      const int end = B.last_seg ? P.H : B.Y1;
      put_row<CHK>(Ra, 2 * k - 1, CHK ? (2 * k - 1 - end) >> 31 : -1);
      put_row<CHK>(X, 2 * k, CHK ? (2 * k - end) >> 31 : -1);
    }
  }
  // A copy in a register of its own: without it the previous high row keeps
  // the slot's registers, and the slot's next load needs others.
  __device__ __forceinline__ static void copy(uint32_t &to, uint32_t from) {
    asm volatile("v_mov_b32 %0, %1" : "=v"(to) : "v"(from));
  }
  // Ends the use of a ring slot: what read it stays above this point and its
  // next load below (a load moved past its predecessor's use would need
  // registers of its own, and a copy at the loop's end that waits for it).
  template <int n> __device__ __forceinline__ static void free_regs(uint32_t (&a)[n], uint32_t (&b)[n], uint32_t &c) {
#pragma unroll
    for (int j = 0; j < n; ++j) asm volatile("" : "+v"(a[j]), "+v"(b[j]));
    asm volatile("" : "+v"(c));
    __builtin_amdgcn_sched_barrier(0);
  }

  template <int S, bool CHK> __device__ __forceinline__ void unit(int u) {
    if constexpr (CHK) vedge = U * (u + 1) > P.H;
    constexpr int slot = S % Q<L>;
    uint32_t ll[NP<L>];
#pragma unroll
    for (int j = 0; j < NP<L>; ++j) ll[j] = F0[slot][j];
    realign_ll(ll, u);
    decrypt(ll, u);
#pragma unroll
    for (int j = 0; j < NP<L>; ++j) asm volatile("" : "+v"(ll[j]));
    __builtin_amdgcn_sched_barrier(0);
    F0[slot] = next_ll(u + Q<L>);
    step<L, 0, S, CHK>(u, ll);
  }
  __device__ __forceinline__ void decrypt(uint32_t (&ll)[NP<L>], int k) const {
    if (!P.use_aes) return;
    typedef uint32_t u32_h __attribute__((aligned(2)));
    const char *p = reinterpret_cast<const char *>(ks.ks) + ks.row(P, min(k, P.hdim[L] - 1)) + ks_off;
    if constexpr (M<L> == 1) {
      ll[0] ^= *reinterpret_cast<const uint16_t *>(p);
    } else {
#pragma unroll
      for (int j = 0; j < NP<L>; ++j) ll[j] ^= reinterpret_cast<const u32_h *>(p)[j];
    }
  }

  // First step of a segment (step k of level l, k = NS u0): the even row only.
  template <int l> __device__ __forceinline__ void init(int u0, const uint32_t (&ll)[NP<l>]) {
    constexpr int Np = NP<l>, Rl = R<l>;
    const int k = NS<l> * u0, N = P.hdim[l - 1];
    auto &Dv = Dp<l>();
    auto &Xv = Xp<l>();
    uint32_t Sv[Rl], Dq[Rl];
#pragma unroll
    for (int j = 0; j < Np; ++j) {
      Sv[j] = ll[j];
      Sv[Np + j] = Ih<l>()[j];
      Dq[j] = Il<l>()[0][j];
      Dq[Np + j] = Ix<l>()[0][j];
      Dv[j] = Il<l>()[1][j];
      Dv[Np + j] = Ix<l>()[1][j];
    }
    if constexpr (GEN) {
      realign_hl<l>(Sv, k);
      realign_d<l>(Dq, k - 1);
      realign_d<l>(Dv, k);
      inside<l>(Sv, Dq);
      inside<l>(Dv, Dv);
    }
    check(Sv);
    check(Dq);
    check(Dv);
    if (2 * k + 1 >= N) {  // (k = 0 only where the level is one row, without details)
#pragma unroll
      for (int t = 0; t < Rl; ++t) Dv[t] = N == 1 ? 0u : Dq[t];
    }
    if (k == 0) {  // d(-1) = d(1)
#pragma unroll
      for (int t = 0; t < Rl; ++t) Dq[t] = Dv[t];
    }
#pragma unroll
    for (int t = 0; t < Rl; ++t) Xv[t] = pk_sub(Sv[t], pk_sra(pk_add(pk_add(Dq[t], Dv[t]), 0x00020002u), 2));
    if constexpr (l > 1) {
      uint32_t la[NP<l - 1>];
      to_ll<l>(Xv, la);
      init<l - 1>(u0, la);
    } else {
      put_row<true>(Xv, 2 * k, -1);
    }
  }
  template <int l> __device__ __forceinline__ void init_loads(int u0) {
    const int k = NS<l> * u0;
    Ih<l>() = load_hl<l>(k);
    load_d<l>(k - 1, Il<l>()[0], Ix<l>()[0]);
    load_d<l>(k, Il<l>()[1], Ix<l>()[1]);
  }
  template <int l> __device__ __forceinline__ void ring_loads(int u0) {
    ring_start<l>(NS<l> * u0 + 1);
#pragma unroll
    for (int q = 0; q < Q<l>; ++q) {
      next_rows<l>(NS<l> * u0 + 1 + q, Fh<l>()[q], Fl<l>()[q], Fx<l>()[q]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // Issues the loads of the first rows.
  __device__ __forceinline__ void start() {
    c0 = B.cbase + lane * C1;
    redge = c0 + C1 == P.W;
    const int u0 = B.Y0 >> L;
    ulast = (B.Y1 + U - 1) >> L;
    I0 = load_ll(u0);
    if constexpr (L >= 4) init_loads<4>(u0);
    if constexpr (L >= 3) init_loads<3>(u0);
    if constexpr (L >= 2) init_loads<2>(u0);
    init_loads<1>(u0);
    __builtin_amdgcn_sched_barrier(0);
    last_h[L] = min(ulast, P.hdim[L] - 1);
    pLL = uniform_ptr(reinterpret_cast<const char *>(llin + int64_t(min(u0 + 1, last_h[L])) * P.wdim[L]));
#pragma unroll
    for (int q = 0; q < Q<L>; ++q) F0[q] = next_ll(u0 + 1 + q);
    if constexpr (L >= 4) ring_loads<4>(u0);
    if constexpr (L >= 3) ring_loads<3>(u0);
    if constexpr (L >= 2) ring_loads<2>(u0);
    ring_loads<1>(u0);
  }

  // Streams the rectangle; false when a value outside [-4096, 4095] was read
  // (the packed results are then not trusted).
  __device__ __forceinline__ bool run() {
    constexpr int ES = U8OUT ? 1 : 2;
    const int u0 = B.Y0 >> L, u1 = ulast;
    const bool own = c0 >= B.X0 && (B.last_win || c0 < B.X1);
    so = own ? uint32_t(c0) * ES : kNoLane;
    prow = static_cast<char *>(out) + int64_t(B.Y0) * P.W * ES;
    ks_off = 2 * (min(c0 >> L, ks.cl1 - 1) - ks.cl0);
    chk = 0;
    uint32_t ll[NP<L>];
#pragma unroll
    for (int j = 0; j < NP<L>; ++j) ll[j] = I0[j];
    realign_ll(ll, u0);
    decrypt(ll, u0);
    init<L>(u0, ll);
    // The first unit is code of its own: what it leaves in flight is what a
    // trip of the loop does, and the loop's waits are counted for that.
    unit<0, true>(u0 + 1);
    int u = u0 + 2;
    // whole trips of units away from the last rows (of the image: steps ahead
    // are clamped; of the segment: its last row belongs to the next one)
    const int end = min(u1, P.H / U);
#pragma unroll 1
    for (; u + UPL <= end; u += UPL) trip<false>(u, u1);
#pragma unroll 1
    for (; u <= u1; u += UPL) trip<true>(u, u1);
    return __builtin_amdgcn_ballot_w64((chk & kOutside) != 0 && c0 < P.W) == 0;
  }
  // UPL units; a checked trip ends with the segment's last unit.
  template <bool CHK> __device__ __forceinline__ void trip(int u, int u1) {
    unit<1, CHK>(u);
    if constexpr (UPL >= 2) {
      if (CHK && u + 1 > u1) return;
      unit<2, CHK>(u + 1);
    }
    if constexpr (UPL >= 4) {
      if (CHK && u + 2 > u1) return;
      unit<3, CHK>(u + 2);
      if (CHK && u + 3 > u1) return;
      unit<4, CHK>(u + 3);
    }
  }
};

// Whether a wavefront needs the general form.
template <int L, int C1, bool TAIL, class SP>
__device__ __forceinline__ bool inv_is_general(SP &G, const InvRect &B) {
  if ((B.cbase + 64 * C1 > G.W && G.W % C1 != 0) || G.hdim[L - 1] < 2) return true;
  return !TAIL && B.last_seg && G.n_valid < int64_t(G.H) * G.W;
}

// One wavefront's rectangle.  `tables` makes the AES tables and keys of the
// workgroup ready (every wavefront of it passes there, also one without a
// rectangle); the first rows are in flight meanwhile.
template <int L, int C1, bool U8OUT, bool TAIL, class SP, class Tables>
__device__ __forceinline__ void inv_rect(SP &G, int wave, const int16_t *llin, const int16_t *pub,
                                         void *out, uint32_t *lds, const uint32_t *te,
                                         const uint32_t *kw, int lane, const Tables &tables) {
  const bool live = wave < G.n_waves;
  const InvRect B(G, live ? wave : 0);
  const bool general = inv_is_general<L, C1, TAIL>(G, B);
  const InvKeys<L, C1> ks(G, B, lds, B.Y0 >> L);
  InvWavePk<L, C1, U8OUT, false, TAIL, SP> w{G, B, llin, pub, out, ks, lane};
  if (live && !general) w.start();
  if (G.use_aes) tables();
  if (!live) return;
  const int kend = min(G.hdim[L], (B.Y1 + G.halo_b) >> L);
  if (G.use_aes) {
    ks.fill(G, lds, kend, te, kw, lane);
    wave_lds_sync();
  }
  bool ok = false;
  if (general) {
    // (fragments of fewer values than a lane reads: the exact stream)
    if (G.off_hh[1] + int64_t(G.hdim[0] - G.hdim[1]) * (G.wdim[0] - G.wdim[1]) >= C1 / 2 &&
        int64_t(G.hdim[L]) * G.wdim[L] >= max(1, C1 >> L)) {
      InvWavePk<L, C1, U8OUT, true, TAIL, SP> g{G, B, llin, pub, out, ks, lane};
      g.start();
      ok = g.run();
    }
  } else {
    ok = w.run();
  }
  if (ok) return;
  // redone from one LL row further up, after the stores so far
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
  const InvKeys<L, C1> ks32(G, B, lds, max(0, (B.Y0 >> L) - 1));
  if (G.use_aes) {
    ks32.fill(G, lds, kend, te, kw, lane);
    wave_lds_sync();
  }
  InvWave<L, C1, U8OUT, SP> x{G, B, llin, pub, out, ks32, lane};
  x.run();
}

}  // namespace dwtfrag
