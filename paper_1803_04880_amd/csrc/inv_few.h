// Inverse streams of views of few rows (one LL row).
//
// As in the forward (fwd_few.h), a unit of the streaming kernel is 2^L rows
// whatever the view has, and levels of one row take its general form.  Here a
// window's band rows come into LDS, every lane's words its own, and are
// inverted level by level, in loops over the rows there are.  The same packed
// arithmetic and the same check: a window that holds a value outside its range
// is redone in 32 bits.
#pragma once

#include "inv.h"

namespace dwtfrag {

// GEN: widths that cut a lane's columns, as in the streaming kernel.
template <int L, int C1, bool U8OUT, bool GEN, class SP>
struct InvFew : InvWavePk<L, C1, U8OUT, GEN, !GEN, SP> {
  using Base = InvWavePk<L, C1, U8OUT, GEN, !GEN, SP>;
  template <int l> static constexpr int NP = Base::template NP<l>;
  template <int l> static constexpr int R = Base::template R<l>;
  template <int l> using Words = typename Base::template Words<l>;
  static constexpr int kBatch = 4;  // rows of each band in flight

  // rows of level l: LL, HL, LH and HH rows k side by side, the levels one
  // after the other; first[l] words of a lane before level l's
  uint32_t *rows;  // this lane's words: word j at rows[64 * j]
  int first[L + 2];

  __device__ __forceinline__ InvFew(SP &P, const InvRect &B, const int16_t *llin, const int16_t *pub,
                                    void *out, const InvKeys<L, C1> &ks, int lane, uint32_t *rows_)
      : Base(P, B, llin, pub, out, ks, lane), rows(rows_) {
    first[1] = 0;
#pragma unroll
    for (int l = 1; l <= L; ++l) first[l + 1] = first[l] + inv_few_words(C1, l, P.hdim[l]);
  }

  template <int l> __device__ __forceinline__ uint32_t &word(int k, int band, int j) const {
    return rows[64 * (first[l] + (4 * k + band) * NP<l> + j)];
  }

  // Band rows of level l.
  template <int l> __device__ __forceinline__ void fill() {
    const int n = this->P.hdim[l];
#pragma unroll 1
    for (int k0 = 0; k0 < n; k0 += kBatch) {
      Words<l> h[kBatch], lo[kBatch], hi[kBatch];
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        h[i] = this->template load_hl<l>(k0 + i);
        lo[i] = hi[i] = h[i];
        if (this->P.hdim[l - 1] > n) this->template load_d<l>(k0 + i, lo[i], hi[i]);
      }
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        if (k0 + i >= n) break;
#pragma unroll
        for (int j = 0; j < NP<l>; ++j) {
          word<l>(k0 + i, 1, j) = h[i][j];
          word<l>(k0 + i, 2, j) = lo[i][j];
          word<l>(k0 + i, 3, j) = hi[i][j];
        }
      }
    }
  }

  // Row i of the level-(l-1) grid: the LL row of the level below, or an output
  // row (they come in order).
  template <int l> __device__ __forceinline__ void emit(const uint32_t (&x)[R<l>], int i) {
    if constexpr (l > 1) {
      uint32_t la[NP<l - 1>];
      this->template to_ll<l>(x, la);
#pragma unroll
      for (int j = 0; j < NP<l - 1>; ++j) word<l - 1>(i, 0, j) = la[j];
    } else {
      this->template put_row<true>(x, i, -1);
    }
  }

  template <int l> __device__ __forceinline__ void level() {
    constexpr int Np = NP<l>, Rl = R<l>;
    const int N = this->P.hdim[l - 1], n = this->P.hdim[l];
    uint32_t Dv[Rl], Xv[Rl];
#pragma unroll
    for (int t = 0; t < Rl; ++t) { Dv[t] = 0; Xv[t] = 0; }
#pragma unroll 1
    for (int k = 0; k < n; ++k) {
      uint32_t Sv[Rl], Dn[Rl], X[Rl], Ra[Rl];
#pragma unroll
      for (int j = 0; j < Np; ++j) {
        Sv[j] = word<l>(k, 0, j);
        Sv[Np + j] = word<l>(k, 1, j);
        Dn[j] = word<l>(k, 2, j);
        Dn[Np + j] = word<l>(k, 3, j);
      }
      if constexpr (GEN) {
        this->template realign_hl<l>(Sv, k);
        this->template realign_d<l>(Dn, k);
        this->template inside<l>(Sv, Dn);
      }
      this->check(Sv);
      if (2 * k + 1 < N) {
        this->check(Dn);
      } else {  // d(N) = d(N-2); a level of one row has no details
#pragma unroll
        for (int t = 0; t < Rl; ++t) Dn[t] = Dv[t];
      }
#pragma unroll
      for (int t = 0; t < Rl; ++t) {
        const uint32_t prev = k == 0 ? Dn[t] : Dv[t];  // d(-1) = d(1)
        X[t] = pk_sub(Sv[t], pk_sra(pk_add(pk_add(prev, Dn[t]), 0x00020002u), 2));
        Ra[t] = pk_add(Dv[t], pk_sra(pk_add(Xv[t], X[t]), 1));
        Dv[t] = Dn[t];
        Xv[t] = X[t];
      }
      if (k > 0) emit<l>(Ra, 2 * k - 1);
      emit<l>(X, 2 * k);
    }
    if (N % 2 == 0) {  // x(N) = x(N-2)
      uint32_t Ra[Rl];
#pragma unroll
      for (int t = 0; t < Rl; ++t) Ra[t] = pk_add(Dv[t], Xv[t]);
      emit<l>(Ra, N - 1);
    }
  }

  // The loads, before the keystream is there.
  __device__ __forceinline__ void start() {
    this->c0 = this->B.cbase + this->lane * C1;
    this->redge = this->c0 + C1 == this->P.W;
    this->ulast = 1;
    this->I0 = this->load_ll(0);
    fill<1>();
    if constexpr (L >= 2) fill<2>();
    if constexpr (L >= 3) fill<3>();
    if constexpr (L >= 4) fill<4>();
  }
  __device__ __forceinline__ bool run() {
    constexpr int ES = U8OUT ? 1 : 2;
    const bool own = this->c0 >= this->B.X0 && (this->B.last_win || this->c0 < this->B.X1);
    this->so = own ? uint32_t(this->c0) * ES : Base::kNoLane;
    this->prow = static_cast<char *>(this->out);
    this->ks_off = 2 * (min(this->c0 >> L, this->ks.cl1 - 1) - this->ks.cl0);
    this->chk = 0;
    uint32_t ll[NP<L>];
#pragma unroll
    for (int j = 0; j < NP<L>; ++j) ll[j] = this->I0[j];
    this->realign_ll(ll, 0);
    this->decrypt(ll, 0);
#pragma unroll
    for (int j = 0; j < NP<L>; ++j) word<L>(0, 0, j) = ll[j];
    if constexpr (L >= 4) level<4>();
    if constexpr (L >= 3) level<3>();
    if constexpr (L >= 2) level<2>();
    level<1>();
    return __builtin_amdgcn_ballot_w64((this->chk & Base::kOutside) != 0 && this->c0 < this->P.W) == 0;
  }
};

// LDS words of a wavefront's keystream: one row, and a block that lanes past
// its end may read.
template <int L, int C1> constexpr int kInvFewKeys = (64 * C1 / (8 << L) + 3) * 4;

// One wavefront's window, as fwd_few.
template <int L, int C1, bool U8OUT, bool GEN, class SP, class Tables>
__device__ __forceinline__ void inv_few(SP &P, int wave, const int16_t *llin, const int16_t *pub, void *out,
                                        uint32_t *lds_ks, uint32_t *rows, const uint32_t *te, const uint32_t *kw,
                                        int lane, const Tables &tables) {
  const InvRect B(P, wave);
  const InvKeys<L, C1> ks(P, B, lds_ks, 0);
  InvFew<L, C1, U8OUT, GEN, SP> w(P, B, llin, pub, out, ks, lane, rows + lane);
  // (fragments of fewer values than a lane reads: the exact stream)
  const bool packed = P.off_hh[1] + int64_t(P.hdim[0] - P.hdim[1]) * (P.wdim[0] - P.wdim[1]) >= C1 / 2 &&
                      int64_t(P.hdim[L]) * P.wdim[L] >= max(1, C1 >> L);
  if (packed) w.start();
  if (P.use_aes) {
    tables();
    wave_lds_sync();
    ks.fill(P, lds_ks, 1, te, kw, lane);
    wave_lds_sync();
  }
  if (packed && w.run()) return;
  // redone after the stores so far
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
  InvWave<L, C1, U8OUT, SP> x{P, B, llin, pub, out, ks, lane};
  x.run();
}

}  // namespace dwtfrag
