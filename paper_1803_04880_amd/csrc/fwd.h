// Forward path: fused multi-level 5/3 lifting with band scatter and the
// counter-mode encryption of the last LL band, as one streaming kernel.
//
// Ch. 5 section 5.1.1: each level runs the horizontal pass (eqs. (5.1)-(5.2)
// along rows), then the vertical pass, and the next level transforms LL only.
//
// One wavefront owns a rectangle of the level-0 grid (a column window times a
// short row segment) and streams the rows of its window top to bottom in
// units of 2^L rows, all in registers: unit v takes rows 2^L v - 1 ..
// 2^L v + 2^L - 2, so that at every level its rows form whole (odd, even)
// pairs, and low / high row k of level l come out at a place of the code
// that is known at compile time.  A pair completes low row k and high row k;
// detail rows are stored, low rows go straight into the next level's
// horizontal pass.  The keystream of the rectangle's LL elements does not
// depend on the data: it is computed into LDS while the first rows are in
// flight, and the LL rows are XORed with it on their way out.
//
// What bounds it is HBM, and before that the memory system's reordering:
// loads and stores share one in-order counter (vmcnt), so a wait for a row
// must not sit behind stores whose number the compiler cannot count.  The
// unit is therefore straight-line code: every band row is stored by one
// buffer store without a branch (rows that are not owned get a descriptor of
// zero records, lanes that are not owned an offset past its end; the
// hardware drops both), and the next rows' loads are re-issued into the
// registers that the unit frees.  Short segments in the order of the image
// keep the bytes in flight together; the rows a segment recomputes above and
// below its own cost less than the long streams did.  Measured against a
// wavefront per long segment with LDS queues between the levels, which
// waited for its own stores every batch: 256 MiB at three levels 231 -> 177
// us (4.6 TB/s), 16 MiB 46.5 -> 18.4, 12 MB of width 3001 at two levels 65 ->
// 25; at 16 MiB, where a wavefront has a SIMD to itself, it issues for 61% of
// its 18 us.
#pragma once

#include "lift.h"
#include "pack.h"

namespace dwtfrag {

// A wavefront's rectangle and window.
struct FwdRect {
  int win, seg;
  int X0, X1, Y0, Y1;   // owned rectangle (level 0), X1 / Y1 exclusive
  int cbase;            // first column of the window
  bool last_win, last_seg;

  template <class SP> __device__ __forceinline__ FwdRect(SP &G, int wave) {
    win = wave % G.n_win;
    seg = wave / G.n_win;
    last_win = (win == G.n_win - 1);
    last_seg = (seg == G.n_seg - 1);
    X0 = win * G.own_w;
    X1 = last_win ? G.W : X0 + G.own_w;
    Y0 = seg_start(G, seg);
    Y1 = last_seg ? G.H : seg_start(G, seg + 1);
    cbase = (win == 0) ? 0 : X0 - G.halo_l;
  }
};

// 16-byte keystream blocks that a row of the rectangle's LL elements can touch.
template <class SP> __device__ __forceinline__ int fwd_ks_blocks(SP &G, const FwdRect &B, int L) {
  const int cols = (B.last_win ? G.wdim[L] : min(G.wdim[L], B.X1 >> L)) - (B.X0 >> L);
  return ((2 * cols + 30) >> 4);
}

// GEN: windows whose right end cuts a lane's columns, and without TAIL
// wavefronts that read the view's partial last row: per-lane edge masks, cut
// lanes stored in pieces, checked loads.  All others run the plain form, where
// an edge of the row can only lie at a lane's boundary.
// TAIL: the kernels of views with a partial last row.  Their plain form checks
// for that row by itself: the general one takes twice as long a row, and a
// launch lasts as long as its last segment (16 MiB of width 4088, three levels
// 37.0 -> 21.3 us).  Kernels of whole views stay without the checks, which
// cost 6% (16 MiB of width 4096 18.3 -> 19.5 us).
template <int L, int C1, bool U8IN, bool GEN, bool TAIL, class SP>
struct FwdWave {
  template <int l> static constexpr int M = (C1 >> (l - 1)) / 2;  // evens per lane at level l
  template <int l> static constexpr int NP = Pk<M<l>>::P;         // packed regs per parity
  template <int l> static constexpr int R = 2 * NP<l>;            // packed regs per row
  static constexpr int U = 1 << L;                                // rows per unit
  static constexpr int RB = U8IN ? C1 : 2 * C1;                   // input bytes per lane and row
  static constexpr int RW = RB / 4;                               // ... in dwords
  static constexpr int PF = RW > 4 || (GEN && C1 == 16) ? 4 : 8;  // rows in flight per lane
  static constexpr int UPL = PF > U ? PF / U : 1;                 // units per loop trip

  SP &G;
  const FwdRect &B;
  const void *in;
  const uint32_t *ks;     // keystream of the LL rows in LDS (use_aes)
  int16_t *llout;         // LL output
  int lane;
  int c0;                 // level-0 column of this lane's first sample
  uint32_t voff;          // byte offset of this lane's columns in an input row
  bool redge;             // the row ends with this lane's last column
  int vedge;              // the unit touches the first or last rows of a level
  // -1 where the unit's pairs but the first are owned, else 0 (a sign bit, not
  // a comparison: those end up in vector registers)
  int keep1;
  int rlast;              // last row streamed
  int tail_last;          // last_col of the view's last row
  uint32_t q[PF][RW];     // rows in flight

  // per-level registers: previous even row, previous high row
  uint32_t E1[R<1>], D1[R<1>];
  uint32_t E2[L >= 2 ? R<2> : 1], D2[L >= 2 ? R<2> : 1];
  uint32_t E3[L >= 3 ? R<3> : 1], D3[L >= 3 ? R<3> : 1];
  uint32_t E4[L >= 4 ? R<4> : 1], D4[L >= 4 ? R<4> : 1];
  char *pHL[L + 1], *pLH[L + 1];   // the band rows of the next pair of each level
  int64_t dHH[L + 1];              // HH row - HL row (bytes)
  uint32_t so[L + 1];              // this lane's byte offset in a band row, or past its end

  template <int l> __device__ __forceinline__ auto &E() {
    if constexpr (l == 1) return E1; else if constexpr (l == 2) return E2;
    else if constexpr (l == 3) return E3; else return E4;
  }
  template <int l> __device__ __forceinline__ auto &D() {
    if constexpr (l == 1) return D1; else if constexpr (l == 2) return D2;
    else if constexpr (l == 3) return D3; else return D4;
  }

  // ---- input rows --------------------------------------------------------
  // Row r; rows above the view are mirrored, which whole-sample symmetry about
  // row 0 makes exact at every level, rows below the segment's last one are
  // never used.
  __device__ __forceinline__ void load_row(int r, uint32_t (&w)[RW]) const {
    r = min(r < 0 ? -r : r, rlast);
    const int64_t at = int64_t(r) * G.W;
    const char *rowp = static_cast<const char *>(in) + at * (U8IN ? 1 : 2);
    if constexpr (GEN) {
      if (G.n_valid < C1) {  // less than a lane reads: one by one
        load_tiny(rowp, at, w);
        return;
      }
      // lanes past the view's end read its last samples, and the row's use
      // shifts them into place (realign)
      const int last = last_col(at), base = min(last, 0);
      load_at(rowp + base * ES, uint32_t((min(c0, last) - base) * ES), w);
    } else if constexpr (!TAIL) {
      load_at(rowp, voff, w);
    } else {  // the same for the last row
      const bool tail = r == G.H - 1;
      load_at(rowp + (tail ? min(tail_last, 0) * ES : 0),
              min(voff, tail ? uint32_t(max(tail_last, 0) * ES) : 0x7FFFFFFFu), w);
    }
  }
  static constexpr int ES = U8IN ? 1 : 2;
  __device__ __forceinline__ int last_col(int64_t at) const { return last_read_col(G.n_valid, at, C1); }
  __device__ __forceinline__ void load_tiny(const char *rowp, int64_t at, uint32_t (&w)[RW]) const {
#pragma unroll
    for (int i = 0; i < RW; ++i) w[i] = 0;
#pragma unroll 1
    for (int t = C1 - 1; t >= 0; --t) {
#pragma unroll
      for (int i = RW - 1; i > 0; --i) w[i] = __builtin_amdgcn_alignbit(w[i], w[i - 1], 32 - 8 * ES);
      w[0] <<= 8 * ES;
      if (c0 + t < G.W && at + c0 + t < G.n_valid) {
        if constexpr (U8IN) w[0] |= ((gptr<const uint8_t>)glob(rowp))[c0 + t];
        else w[0] |= ((gptr<const uint16_t>)glob(rowp))[c0 + t];
      }
    }
  }
  // Row r as loaded -> its samples in place, zeros past the view's end.
  __device__ __forceinline__ void realign(int r, uint32_t (&w)[RW]) const {
    r = min(r < 0 ? -r : r, rlast);
    int last;
    if constexpr (GEN) {
      last = last_col(int64_t(r) * G.W);
      if (last >= G.W || G.n_valid < C1) return;
    } else {
      if (r != G.H - 1) return;
      last = tail_last;
    }
    const int sh = read_shift(c0, last, C1) * ES;  // bytes
#pragma unroll
    for (int b = 1; b <= 4 * RW; b *= 2)
#pragma unroll
      for (int i = 0; i < RW; ++i) {
        const int up = b / 4;
        const uint32_t v = b < 4 ? __builtin_amdgcn_alignbit(i + 1 < RW ? w[i + 1 < RW ? i + 1 : i] : 0u, w[i], 8 * (b & 3))
                                 : (i + up < RW ? w[i + up < RW ? i + up : i] : 0u);
        w[i] = (sh & b) ? v : w[i];
      }
  }
  // C1 samples at byte off of the row at rowp.
  __device__ __forceinline__ void load_at(const char *rowp, uint32_t off, uint32_t (&w)[RW]) const {
    // (the address stays in scalar registers: the lane's offset is all of its
    // vector part)
    const gptr<const char> src = glob(uniform_ptr(rowp));
    if constexpr (RW == 2) {
      const u32x2 v = *(gptr<const u32x2_u>)(src + off);
      w[0] = v.x; w[1] = v.y;
    } else {
#pragma unroll
      for (int i = 0; i < RW; i += 4) {
        const u32x4 v = *(gptr<const u32x4_u>)(src + off + 4u * i);
        w[i] = v.x; w[i + 1] = v.y; w[i + 2] = v.z; w[i + 3] = v.w;
      }
    }
  }

  // Input row -> even / odd packed registers of level 1.
  __device__ __forceinline__ void unpack(const uint32_t (&w)[RW], uint32_t (&Ein)[NP<1>],
                                         uint32_t (&Oin)[NP<1>]) const {
    if constexpr (U8IN) {
#pragma unroll
      for (int j = 0; j < NP<1>; ++j) {
        Ein[j] = __builtin_amdgcn_perm(0u, w[j], 0x0C020C00u);  // (b0, b2)
        Oin[j] = __builtin_amdgcn_perm(0u, w[j], 0x0C030C01u);  // (b1, b3)
      }
    } else {
#pragma unroll
      for (int j = 0; j < NP<1>; ++j) {
        Ein[j] = lo_halves(w[2 * j], w[2 * j + 1]);
        Oin[j] = hi_halves(w[2 * j], w[2 * j + 1]);
      }
    }
  }

  // Ends the use of a ring slot: the unpacking stays above this point and the
  // slot's next load below it.  With one moved past the other the load would
  // need registers of its own, and a copy at the loop's end that waits for it.
  __device__ __forceinline__ static void free_slot(uint32_t (&Ein)[NP<1>], uint32_t (&Oin)[NP<1>]) {
#pragma unroll
    for (int j = 0; j < NP<1>; ++j) asm volatile("" : "+v"(Ein[j]), "+v"(Oin[j]));
    __builtin_amdgcn_sched_barrier(0);
  }

  // ---- band rows ---------------------------------------------------------
  // M values of this lane at offset so[l] of a band row of `cols` columns.
  template <int l>
  __device__ __forceinline__ void store_row(char *row, int keep, int cols, const uint32_t *V) const {
    constexpr int Mv = M<l>;
    // (the descriptor is uniform; said so, lest the compiler loop over lanes)
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(
        uniform_ptr(row), 0, __builtin_amdgcn_readfirstlane((2 * cols) & keep), 0x00027000);
    uint32_t off = so[l];
    if constexpr (GEN && Mv > 1) {
      // a lane that the row's end cuts stores its first nv values as one
      // vector of 4, 2 and 1 each, where nv has that bit
      const int nv = cols - (c0 >> l);
      const bool cut = nv > 0 && nv < Mv && off != kNoLane;
      if constexpr (Mv >= 8)
        __builtin_amdgcn_raw_buffer_store_b64(u32x2{V[0], V[1]}, rsrc, cut && (nv & 4) ? off : kNoLane, 0, kStoreAux);
      if constexpr (Mv >= 4) {
        const uint32_t two = Mv >= 8 ? ((nv & 4) ? V[2 % NP<l>] : V[0]) : V[0];
        __builtin_amdgcn_raw_buffer_store_b32(two, rsrc, cut && (nv & 2) ? off + 2 * (nv & 4) : kNoLane, 0, kStoreAux);
      }
      uint32_t one = V[0];
#pragma unroll
      for (int i = 1; i < NP<l>; ++i) one = (nv >> 1) == i ? V[i] : one;
      __builtin_amdgcn_raw_buffer_store_b16(uint16_t(one), rsrc, cut && (nv & 1) ? off + 2 * (nv - 1) : kNoLane, 0, kStoreAux);
      if (nv < Mv) off = kNoLane;
    }
    if constexpr (Mv == 8)
      __builtin_amdgcn_raw_buffer_store_b128(u32x4{V[0], V[1], V[2], V[3]}, rsrc, off, 0, kStoreAux);
    else if constexpr (Mv == 4)
      __builtin_amdgcn_raw_buffer_store_b64(u32x2{V[0], V[1]}, rsrc, off, 0, kStoreAux);
    else if constexpr (Mv == 2)
      __builtin_amdgcn_raw_buffer_store_b32(V[0], rsrc, off, 0, kStoreAux);
    else
      __builtin_amdgcn_raw_buffer_store_b16(uint16_t(V[0]), rsrc, off, 0, kStoreAux);
  }
  static constexpr uint32_t kNoLane = 0x80000000u;
  static constexpr int kStoreAux = 2;  // nt

  // ---- one level ---------------------------------------------------------
  // Horizontal pass of a row of level l, in place.
  template <int l>
  __device__ __forceinline__ void lift_row(uint32_t (&Ein)[NP<l>], uint32_t (&Oin)[NP<l>],
                                           uint32_t (&x)[R<l>]) const {
    constexpr int Np = NP<l>;
    if constexpr (GEN) {
      hfwd_pk_any<M<l>>(Ein, Oin, c0 >> (l - 1), G.wdim[l - 1], true);
    } else {
      hfwd_pk_lanes<M<l>>(Ein, Oin, redge);
    }
#pragma unroll
    for (int j = 0; j < Np; ++j) { x[j] = Ein[j]; x[Np + j] = Oin[j]; }
  }

  // Lifted row J of unit v of level l: an input row (S: the unit's place in
  // the loop trip, which fixes the ring slot; 0 is the segment's first unit),
  // or low row J of level l - 1.
  template <int l, int J, int S, bool CHK>
  __device__ __forceinline__ void row(int v, uint32_t (&x)[R<l>]) {
    uint32_t Ein[NP<l>], Oin[NP<l>];
    if constexpr (l == 1) {
      constexpr int slot = (kWarm<0> + S * U + J) % PF;
      if constexpr (CHK && (GEN || TAIL)) realign(U * v - 1 + J, q[slot]);
      unpack(q[slot], Ein, Oin);
      free_slot(Ein, Oin);
      if constexpr (CHK) {
        load_row(U * v - 1 + J + PF, q[slot]);
      } else {
        load_at(pnext, voff, q[slot]);
        pnext += int64_t(G.W) * (U8IN ? 1 : 2);
      }
    } else {
      uint32_t low[R<l - 1>];
      pair<l - 1, J, S, CHK>(v, low);
      split<l>(low, Ein, Oin);
    }
    lift_row<l>(Ein, Oin, x);
  }

  // The lows of a level l - 1 row -> even / odd packed registers of level l.
  template <int l>
  __device__ __forceinline__ static void split(const uint32_t (&low)[R<l - 1>], uint32_t (&Ein)[NP<l>],
                                               uint32_t (&Oin)[NP<l>]) {
    if constexpr (M<l> >= 2) {
#pragma unroll
      for (int j = 0; j < NP<l>; ++j) {
        Ein[j] = lo_halves(low[2 * j], low[2 * j + 1]);
        Oin[j] = hi_halves(low[2 * j], low[2 * j + 1]);
      }
    } else {
      Ein[0] = low[0];
      Oin[0] = low[0] >> 16;
    }
  }

  // ---- rows above the segment --------------------------------------------
  // Before the first unit, every level needs its previous even row and the
  // levels below the last their previous high row: kWarm<l> low rows of
  // level l (level 0: input rows), each two rows of level l - 1 plus two for
  // the first high row and one even row.  They end just above the first
  // unit's rows and touch no edge but the mirrored top.
  template <int l> static constexpr int kWarm = l == L ? 0 : l + 1 == L ? 1 : 2 * kWarm<(l < L ? l + 1 : l)> + 3;

  // Warm-up row i of level l, lifted.
  template <int l, int i> __device__ __forceinline__ void warm_row(int r0, uint32_t (&x)[R<l>]) {
    uint32_t Ein[NP<l>], Oin[NP<l>];
    if constexpr (l == 1) {
      constexpr int slot = i % PF;
      if constexpr (GEN) realign(r0 + i, q[slot]);
      unpack(q[slot], Ein, Oin);
      free_slot(Ein, Oin);
      load_row(r0 + i + PF, q[slot]);
    } else {
      uint32_t low[R<l - 1>];
      if constexpr (i == 0) warm_init<l - 1>(r0);
      warm_pair<l - 1, i + 1>(r0, low);
      split<l>(low, Ein, Oin);
    }
    lift_row<l>(Ein, Oin, x);
  }
  // Warm-up pair p of level l (the first one only yields the high row).
  template <int l, int p> __device__ __forceinline__ void warm_pair(int r0, uint32_t (&low)[R<l>]) {
    uint32_t o[R<l>], e[R<l>];
    warm_row<l, 2 * p + 1>(r0, o);
    warm_row<l, 2 * p + 2>(r0, e);
    auto &Ev = E<l>();
    auto &Dv = D<l>();
#pragma unroll
    for (int t = 0; t < R<l>; ++t) {
      const uint32_t dn = pk_predict(o[t], Ev[t], e[t]);
      low[t] = pk_update(Ev[t], Dv[t], dn);
      Dv[t] = dn;
      Ev[t] = e[t];
    }
  }
  template <int l> __device__ __forceinline__ void warm_init(int r0) {
    warm_row<l, 0>(r0, E<l>());
    if constexpr (l < L) {
      uint32_t none[R<l>];
      warm_pair<l, 0>(r0, none);
    }
  }

  // Pair J of unit v at level l: rows (2k+1, 2k+2), k = (U >> l) v - 1 + J.
  // Stores high row k and the HL part of low row k; low row k's lows are
  // returned in low[0 .. NP).  At the first pair d(-1) = d(1); past the last
  // row x(N) = x(N-2), d(N) = d(N-2).
  // CHK: the unit may touch the edges of the image or of the segment.
  template <int l, int J, int S, bool CHK>
  __device__ __forceinline__ void pair(int v, uint32_t (&low)[R<l>]) {
    constexpr int Rl = R<l>, Np = NP<l>;
    const int k = (U >> l) * v - 1 + J;
    auto &Ev = E<l>();
    auto &Dv = D<l>();
    uint32_t o[Rl], e[Rl], dn[Rl];
    row<l, 2 * J, S, CHK>(v, o);
    row<l, 2 * J + 1, S, CHK>(v, e);
    const int N = G.hdim[l - 1];
    if (CHK && vedge && 2 * k + 2 >= N) {
#pragma unroll
      for (int t = 0; t < Rl; ++t) e[t] = Ev[t];
    }
#pragma unroll
    for (int t = 0; t < Rl; ++t) dn[t] = pk_predict(o[t], Ev[t], e[t]);
    if (CHK && vedge) {
      if (2 * k + 1 >= N) {
#pragma unroll
        for (int t = 0; t < Rl; ++t) dn[t] = N == 1 ? 0u : Dv[t];
      }
      if (k <= 0) {
#pragma unroll
        for (int t = 0; t < Rl; ++t) Dv[t] = dn[t];
      }
    }
#pragma unroll
    for (int t = 0; t < Rl; ++t) {
      low[t] = pk_update(Ev[t], Dv[t], dn[t]);
      Dv[t] = dn[t];
      Ev[t] = e[t];
    }
    const int wl = G.wdim[l], wh = G.wdim[l - 1] - wl;
    if constexpr (S > 0 || J > 0) {  // (the first unit's first rows belong to the segment above)
      const int keep = J == 0 ? -1 : keep1;
      const int has_low = CHK ? keep & ((k - G.hdim[l]) >> 31) : -1;
      const int has_high = CHK ? keep & ((k - (N - G.hdim[l])) >> 31) : -1;
      store_row<l>(pLH[l], has_high, wl, dn);
      store_row<l>(pHL[l] + dHH[l], has_high, wh, dn + Np);
      store_row<l>(pHL[l], has_low, wh, low + Np);
      if constexpr (l == L) {
        uint32_t out[Np];
#pragma unroll
        for (int j = 0; j < Np; ++j) out[j] = low[j];
        if (G.use_aes) {
          // keystream bytes of this lane's elements of LL row k (a row's
          // first block starts up to 14 bytes before its first element)
          const int at = (k - (B.Y0 >> L)) * 16 * ks_nb + (2 * (k * (wl & 7) + ks_c0) & 15);
          encrypt(out, has_low ? at : 0);
        }
        store_row<l>(pLL, has_low, wl, out);
      }
    }
    pLH[l] = uniform_ptr(pLH[l] + 2 * int64_t(wl));
    pHL[l] = uniform_ptr(pHL[l] + 2 * int64_t(wh));
    if constexpr (l == L) pLL = uniform_ptr(pLL + 2 * int64_t(wl));
  }

  // XORs this lane's LL elements with the keystream of the row that begins at
  // byte `at`.
  __device__ __forceinline__ void encrypt(uint32_t (&out)[NP<L>], int at) const {
    typedef uint32_t u32_h __attribute__((aligned(2)));
    const char *p = reinterpret_cast<const char *>(ks) + at + ks_off;
    if constexpr (M<L> == 1) {
      out[0] ^= *reinterpret_cast<const uint16_t *>(p);
    } else {
#pragma unroll
      for (int j = 0; j < NP<L>; ++j) out[j] ^= reinterpret_cast<const u32_h *>(p)[j];
    }
  }

  template <int S, bool CHK> __device__ __forceinline__ void unit(int v, int v1) {
    if constexpr (CHK) {
      vedge = v <= 1 || U * (v + 1) - 2 >= G.H;
      keep1 = (v - v1) >> 31;
    }
    uint32_t low[R<L>];
    pair<L, 0, S, CHK>(v, low);
  }

  template <int l> __device__ __forceinline__ void setup_level(int vs) {
    const int wl = G.wdim[l], wh = G.wdim[l - 1] - wl;
    const int bc = c0 >> l;
    const bool lown = bc >= (B.X0 >> l) && (B.last_win || bc < (B.X1 >> l));
    so[l] = lown ? 2u * uint32_t(bc) : kNoLane;
    const int64_t k = int64_t(U >> l) * vs - 1;
    pHL[l] = pub8 + 2 * (G.off_hl[l] + k * wh);
    pLH[l] = pub8 + 2 * (G.off_lh[l] + k * wl);
    dHH[l] = 2 * (G.off_hh[l] - G.off_hl[l]);
    if constexpr (l == L) {
      pLL = reinterpret_cast<char *>(llout) + 2 * (k * wl);
      ks_c0 = B.X0 >> L;
      ks_nb = fwd_ks_blocks(G, B, L);
      ks_off = lown ? 2 * (bc - ks_c0) : 0;
    }
  }
  char *pub8;
  char *pLL;               // the next LL row
  int ks_c0, ks_nb;        // first owned LL column, keystream blocks per row
  int ks_off;              // this lane's bytes in a keystream row

  // Issues the loads of the first rows.
  __device__ __forceinline__ void start() {
    c0 = B.cbase + lane * C1;
    // lanes past the row's end read its last columns (plain form) or the
    // bytes behind it (general form, where they lie inside the view)
    voff = uint32_t(GEN ? c0 : min(c0, G.W - C1)) * (U8IN ? 1u : 2u);
    redge = c0 + C1 == G.W;
    rlast = min(G.H, B.Y1 + U) - 1;
    tail_last = last_col(int64_t(G.H - 1) * G.W);
    const int v0 = B.Y0 >> L;
    const int r0 = U * v0 - 1 - kWarm<0>;  // first warm-up row
    if (v0 > 0) {
#pragma unroll
      for (int i = 0; i < PF; ++i) {
        load_row(r0 + i, q[i]);
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {  // the first segment starts with the unit of row -1
#pragma unroll
      for (int i = 0; i < PF; ++i) {
        load_row(i - 1, q[(kWarm<0> + i) % PF]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }

  // Streams the rectangle.
  __device__ __forceinline__ void run() {
    const int v0 = B.Y0 >> L, v1 = (B.Y1 + U - 1) >> L;
    const int r0 = U * v0 - 1 - kWarm<0>;
    setup_level<1>(v0);
    if constexpr (L >= 2) setup_level<2>(v0);
    if constexpr (L >= 3) setup_level<3>(v0);
    if constexpr (L >= 4) setup_level<4>(v0);
#pragma unroll
    for (int t = 0; t < R<1>; ++t) { E1[t] = 0; D1[t] = 0; }
#pragma unroll
    for (int t = 0; t < (L >= 2 ? R<2> : 1); ++t) { E2[t] = 0; D2[t] = 0; }
#pragma unroll
    for (int t = 0; t < (L >= 3 ? R<3> : 1); ++t) { E3[t] = 0; D3[t] = 0; }
#pragma unroll
    for (int t = 0; t < (L >= 4 ? R<4> : 1); ++t) { E4[t] = 0; D4[t] = 0; }
    if (v0 > 0) warm_init<L>(r0);
    // The first unit is code of its own: what it leaves in flight is what a
    // trip of the loop does, and the loop's waits are counted for the lesser
    // of the two.
    unit<0, true>(v0, v1);
    int v = v0 + 1;
    {
      // whole trips of units that touch no edge, nor does what they prefetch
      // (tail: nor the partial last row; general form: nor rows that a window
      // reaches past the view from)
      const int rvec = GEN ? min(rlast, G.H - 3 - 64 * C1 / G.W) : TAIL ? min(rlast, G.H - 2) : rlast;
      const int end = min(v1, (rvec + 2 - PF) >> L);
      if (v == 1 && v + UPL <= end) {  // (the second unit still holds top rows)
        trip<true>(v, v1);
        v += UPL;
      }
      pnext = static_cast<const char *>(in) + int64_t(U * v - 1 + PF) * G.W * (U8IN ? 1 : 2);
#pragma unroll 1
      for (; v + UPL <= end; v += UPL) trip<false>(v, v1);
    }
#pragma unroll 1
    for (; v <= v1; v += UPL) trip<true>(v, v1);
  }
  // UPL units; a checked trip ends with the segment's last unit.
  template <bool CHK> __device__ __forceinline__ void trip(int v, int v1) {
    unit<1, CHK>(v, v1);
    if constexpr (UPL >= 2) {
      if (CHK && v + 1 > v1) return;
      unit<2, CHK>(v + 1, v1);
    }
    if constexpr (UPL >= 4) {
      if (CHK && v + 2 > v1) return;
      unit<3, CHK>(v + 2, v1);
      if (CHK && v + 3 > v1) return;
      unit<4, CHK>(v + 3, v1);
    }
  }
  const char *pnext;   // the next row to load in unchecked units
};

// Keystream of a wavefront's owned LL rectangle into LDS: the keystream is
// indexed by the byte offset in the LL band, so every 16-byte block that a
// row touches is computed by itself (one shared with a neighbour's rectangle
// by both).  Row r's blocks start at block r * fwd_ks_blocks.
template <int L, class SP>
__device__ __forceinline__ void fwd_keystream(SP &G, const FwdRect &B, uint32_t *ks,
                                              const uint32_t *te, const uint32_t *kw, int lane) {
  const int kr0 = B.Y0 >> L;
  const int kr1 = B.last_seg ? G.hdim[L] : min(G.hdim[L], B.Y1 >> L);
  const int cc0 = B.X0 >> L;
  const int cc1 = B.last_win ? G.wdim[L] : min(G.wdim[L], B.X1 >> L);
  const int nb = fwd_ks_blocks(G, B, L);
  const int total = (kr1 - kr0) * nb;
  // lane work item i = (row kr0 + i / nb, block i % nb of that row); the
  // pair is stepped by 64 items per pass instead of divided each time
  const int step_r = 64 / nb, step_c = 64 % nb;
  int r = lane / nb, c = lane % nb;
#pragma unroll 1
  for (int i = lane; i < total; i += 64) {
    const int64_t e = int64_t(kr0 + r) * G.wdim[L] + cc0;  // the row's first element
    const int64_t b = (e >> 3) + c;
    if (8 * b < e + (cc1 - cc0)) {
      uint32_t w[4];
      counter_block(kw, uint64_t(b), w);
      aes_encrypt(te, kw, w);
      *reinterpret_cast<uint4 *>(ks + 4 * i) = make_uint4(w[0], w[1], w[2], w[3]);
    }
    c += step_c;
    r += step_r;
    if (c >= nb) { c -= nb; ++r; }
  }
}

// Whether a wavefront needs the general form (also where the view holds less
// than a lane reads).
template <int L, int C1, bool TAIL, class SP>
__device__ __forceinline__ bool fwd_is_general(SP &G, const FwdRect &B) {
  const int end = B.cbase + 64 * C1;
  if ((end > G.W && G.W % C1 != 0) || G.n_valid < C1) return true;
  if constexpr (TAIL) return false;
  const int64_t last = int64_t(min(G.H, B.Y1 + (1 << L)) - 1) * G.W;
  return last + min(G.W, end) > G.n_valid;
}

// One wavefront's rectangle.  `tables` makes the AES tables and keys of the
// workgroup ready (every wavefront of it passes there, also one without a
// rectangle); the first rows are in flight meanwhile.
template <int L, int C1, bool U8IN, bool TAIL, class SP, class Tables>
__device__ __forceinline__ void fwd_rect(SP &G, int wave, const void *in, int16_t *pub,
                                         int16_t *llout, uint32_t *ks, const uint32_t *te,
                                         const uint32_t *kw, int lane, const Tables &tables) {
  const bool live = wave < G.n_waves;
  const FwdRect B(G, live ? wave : 0);
  const bool general = fwd_is_general<L, C1, TAIL>(G, B);
  FwdWave<L, C1, U8IN, false, TAIL, SP> w{G, B, in, ks, llout, lane};
  w.pub8 = reinterpret_cast<char *>(pub);
  if (live && !general) w.start();
  if (G.use_aes) tables();
  if (!live) return;
  if (G.use_aes) {
    fwd_keystream<L>(G, B, ks, te, kw, lane);
    wave_lds_sync();
  }
  if (general) {
    FwdWave<L, C1, U8IN, true, TAIL, SP> g{G, B, in, ks, llout, lane};
    g.pub8 = reinterpret_cast<char *>(pub);
    g.start();
    g.run();
  } else {
    w.run();
  }
}

}  // namespace dwtfrag
