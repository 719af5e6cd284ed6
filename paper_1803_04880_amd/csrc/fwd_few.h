// Forward streams of views of few rows (one LL row).
//
// The streaming kernel takes units of 2^L rows, two at least, whatever the
// view has: 32 rows for one, and in the general form twice as long each.  Here
// a wavefront's window comes into LDS whole and is lifted level by level, in
// loops over the rows there are.  Every lane reads and writes its own columns'
// words only, so that nothing is synchronised.  What bounds it is latency: the
// rows arrive in one or two batches, and the rest is a serial chain of about
// half a microsecond a row.
#pragma once

#include "fwd.h"

namespace dwtfrag {

template <int L, int C1, bool U8IN, class SP>
struct FwdFew : FwdWave<L, C1, U8IN, true, false, SP> {
  using Base = FwdWave<L, C1, U8IN, true, false, SP>;
  template <int l> static constexpr int NP = Base::template NP<l>;
  template <int l> static constexpr int R = Base::template R<l>;
  static constexpr int RW = Base::RW;
  static constexpr int kBatch = 8;  // rows in flight

  uint32_t *rows;          // this lane's words: word j of row r at rows[64 * (r * words + j)]

  // The view's rows.
  __device__ __forceinline__ void fill() {
    this->c0 = this->B.cbase + this->lane * C1;
    this->rlast = this->G.H - 1;
#pragma unroll 1
    for (int r0 = 0; r0 < this->G.H; r0 += kBatch) {
      uint32_t w[kBatch][RW];
#pragma unroll
      for (int i = 0; i < kBatch; ++i) this->load_row(r0 + i, w[i]);
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        if (r0 + i >= this->G.H) break;
        this->realign(r0 + i, w[i]);
#pragma unroll
        for (int j = 0; j < RW; ++j) rows[64 * ((r0 + i) * RW + j)] = w[i][j];
      }
    }
  }

  // Row i of level l, lifted: an input row, or low row i of level l - 1.
  template <int l> __device__ __forceinline__ void fetch(int i, uint32_t (&x)[R<l>]) const {
    uint32_t Ein[NP<l>], Oin[NP<l>];
    if constexpr (l == 1) {
      uint32_t w[RW];
#pragma unroll
      for (int j = 0; j < RW; ++j) w[j] = rows[64 * (i * RW + j)];
      this->unpack(w, Ein, Oin);
    } else {
      uint32_t low[R<l - 1>];
#pragma unroll
      for (int j = 0; j < NP<l - 1>; ++j) low[j] = rows[64 * (i * NP<l - 1> + j)];
      Base::template split<l>(low, Ein, Oin);
    }
    this->template lift_row<l>(Ein, Oin, x);
  }

  // Level l: low and high row k from rows 2k .. 2k + 2.  Low rows replace the
  // rows they came from (fewer words, and never ahead of the rows to come).
  template <int l> __device__ __forceinline__ void level() {
    constexpr int Np = NP<l>, Rl = R<l>;
    const auto &G = this->G;
    const int N = G.hdim[l - 1], wl = G.wdim[l], wh = G.wdim[l - 1] - wl;
    uint32_t Ev[Rl], Dv[Rl];
    fetch<l>(0, Ev);
#pragma unroll
    for (int t = 0; t < Rl; ++t) Dv[t] = 0;
#pragma unroll 1
    for (int k = 0; k < G.hdim[l]; ++k) {
      uint32_t e[Rl], dn[Rl], low[Rl];
#pragma unroll
      for (int t = 0; t < Rl; ++t) { e[t] = Ev[t]; dn[t] = Dv[t]; }  // x(N) = x(N-2), d(N) = d(N-2)
      if (2 * k + 1 < N) {
        uint32_t o[Rl];
        fetch<l>(2 * k + 1, o);
        if (2 * k + 2 < N) fetch<l>(2 * k + 2, e);
#pragma unroll
        for (int t = 0; t < Rl; ++t) dn[t] = pk_predict(o[t], Ev[t], e[t]);
        this->template store_row<l>(this->pub8 + 2 * (G.off_lh[l] + int64_t(k) * wl), -1, wl, dn);
        this->template store_row<l>(this->pub8 + 2 * (G.off_hh[l] + int64_t(k) * wh), -1, wh, dn + Np);
      }
#pragma unroll
      for (int t = 0; t < Rl; ++t) {
        low[t] = pk_update(Ev[t], k == 0 ? dn[t] : Dv[t], dn[t]);  // d(-1) = d(1)
        Dv[t] = dn[t];
        Ev[t] = e[t];
      }
      this->template store_row<l>(this->pub8 + 2 * (G.off_hl[l] + int64_t(k) * wh), -1, wh, low + Np);
      if constexpr (l < L) {
#pragma unroll
        for (int j = 0; j < Np; ++j) rows[64 * (k * Np + j)] = low[j];
      } else {
        uint32_t out[Np];
#pragma unroll
        for (int j = 0; j < Np; ++j) out[j] = low[j];
        if (G.use_aes) this->encrypt(out, 2 * this->ks_c0 & 15);
        this->template store_row<l>(reinterpret_cast<char *>(this->llout), -1, wl, out);
      }
    }
  }

  __device__ __forceinline__ void run() {
    this->template setup_level<1>(0);
    if constexpr (L >= 2) this->template setup_level<2>(0);
    if constexpr (L >= 3) this->template setup_level<3>(0);
    if constexpr (L >= 4) this->template setup_level<4>(0);
    level<1>();
    if constexpr (L >= 2) level<2>();
    if constexpr (L >= 3) level<3>();
    if constexpr (L >= 4) level<4>();
  }
};

// LDS words of a wavefront, beside the AES tables and key words.
template <int L, int C1> constexpr int kFwdFewKeys = fwd_ks_words(L, C1) / fwd_ll_rows(L, C1);
template <int L, int C1, bool U8IN> constexpr int kFwdFewRows = 64 * (1 << L) * (U8IN ? C1 / 4 : C1 / 2);

// One wavefront's window; it is its workgroup's only one.  `tables` makes the
// AES tables and keys ready.
template <int L, int C1, bool U8IN, class SP, class Tables>
__device__ __forceinline__ void fwd_few(SP &P, int wave, const void *in, int16_t *pub, int16_t *llout, uint32_t *ks,
                                        uint32_t *rows, const uint32_t *te, const uint32_t *kw, int lane,
                                        const Tables &tables) {
  const FwdRect B(P, wave);
  FwdFew<L, C1, U8IN, SP> w{{P, B, in, ks, llout, lane}};
  w.pub8 = reinterpret_cast<char *>(pub);
  w.rows = rows + lane;
  w.fill();
  if (P.use_aes) {
    tables();
    wave_lds_sync();
    fwd_keystream<L>(P, B, ks, te, kw, lane);
    wave_lds_sync();
  }
  w.run();
}

}  // namespace dwtfrag
