// The adiabatic preconditioner z = F F^T r of one right-hand side inside one
// workgroup (Sec. V A, Eqs. CG_precon, P_change_basis; App. C): a batch item,
// or a small system's solve.
//
// The same three steps as the single-system kernels (fph_precond.h), run by
// one workgroup over the item's whole vector:
//   1. forward transform: for every tile of sites, the twisted half-
//      spectrum DFT over tau, Z_k[i] = (U r)_{2k}, k < H = Ltau/2, through
//      LDS as a Cooley-Tukey split H = H1 H2, into the item's Z workspace;
//   2. for the frequencies k, as many side by side as the workgroup has
//      threads for (bpc_groups), the conjugate series in A^T and then the
//      series in A on block k (cheb_series, one even plaquette per thread,
//      NT >= Q), in place in Z;
//   3. inverse transform of Z into z, with r . z accumulated.
// T is the iteration precision; the tables (bounds, N_P, coefficients,
// twiddles) are per system.
#pragma once

#include "fph_common.h"
#include "fph_precond.h"

namespace fph {

// Preconditioner tables of one system (device pointers).
template <typename T>
struct PcView {
  using T2 = typename Cplx<T>::type;
  const PcInfo* info;   // bounds and series constants
  const int* np;        // N_P(w), w < Ltau
  const T2* coef;       // [H][kNPMax]: c_m(2k)
  const T* dbar;        // [N]
  const T2* tw;         // [H]: e^{-i pi tau / Ltau}
  const T2* W;          // [H]: W_H^k
  const T2* F;          // H1 x H1 then H2 x H2 DFT matrices
  T c4;                 // cosh(dtau t)^4 (joins dbar in the series)
  int H, H1, H2;
  const T2* dense;      // matrices of the longest blocks (k_pc_dense), or nullptr
};

// LDS budgets of the transforms' tiles and of the series' buffers: a workgroup
// alone on its compute unit, and one that shares it (up to four together).
constexpr int kBpcLdsAlone = 112 << 10;
constexpr int kBpcLdsShared = 32 << 10;
__host__ __device__ constexpr int bpc_budget(int nt) { return nt >= 1024 ? kBpcLdsAlone : kBpcLdsShared; }

// Tile width (log2) of the transforms: 32 sites (16 at L = 4), and up to 128 in
// a workgroup alone on its unit, so that each phase of a tile (a round trip to
// memory, two short DFTs) has work for all its waves.
__host__ __device__ inline int bpc_tile_log2(int N, int H, int budget, int elem) {
  int l = N >= 32 ? 5 : 4;
  if (budget >= kBpcLdsAlone)
    while (l < 7 && (2 << l) <= N && 2L * H * (2 << l) * elem <= budget) ++l;
  return l;
}

// LDS (complex values) of the transforms' tables and tiles, and of the series of
// one frequency.
__host__ __device__ inline long bpc_lds_tables(int H1, int H2) {
  return ((long)H1 * H1 + (long)H2 * H2 + (long)H1 * H2 + 1) & ~1L;  // (what follows stays aligned)
}
__host__ __device__ inline long bpc_lds_tf(int H, int lks) { return (2L * H) << lks; }
__host__ __device__ inline long bpc_lds_series(int L) {
  return 2L * (2L * kpm_row_stride(L / 2) * L + kWinPad);
}

// Frequencies whose series run side by side in a workgroup of nt threads
// (elem bytes per complex value): with up to 32 plaquettes one wave each, else
// Q threads each.
constexpr int kBpcWaveQ = 32;
constexpr int kBpcDenseN = 36;  // most sites of a block matrix here
__host__ __device__ inline int bpc_groups(int L, int H, int nt, int budget, int elem) {
  const int Q = L * L / 4;
  const int fit = budget / (int)(bpc_lds_series(L) * elem);
  int G = Q <= kBpcWaveQ ? nt / 64 : nt / Q;
  if (G > fit) G = fit;
  if (G > H) G = H;
  return G < 1 ? 1 : G;
}

// One output of a short DFT over y[j s] (odd lengths; even ones take dft_pair).
template <bool CONJ, typename T2>
FPH_DEVINL T2 dft_one(const T2* fr, const T2* y, int s, int n) {
  T2 acc = T2{0, 0};
#pragma unroll 5
  for (int j = 0; j < n; ++j) {
    if (CONJ) cmacc(acc, fr[j], y[j * s]);
    else cmac(acc, fr[j], y[j * s]);
  }
  return acc;
}

// Step 1 of a tile of 2^lks sites: the H1-point DFTs over n1 of
// X_{n2 + H2 n1}, times W_H^{n2 k1} (all conjugated with CONJ), into
// Y[n2 H1 + k1].
template <typename T, int NT, bool CONJ>
FPH_DEVINL void bpc_step1(const typename Cplx<T>::type* Fl, const typename Cplx<T>::type* Wl,
                          const typename Cplx<T>::type* X, typename Cplx<T>::type* Y, int H1, int H2,
                          int lks) {
  using T2 = typename Cplx<T>::type;
  const int KS = 1 << lks, H = H1 * H2, s1 = H2 << lks;
  auto post = [&](T2 a, int m) {
    return CONJ ? cmulc<T2, T>(a, Wl[m]) : cmul<T2, T>(a, Wl[m]);
  };
  if (H1 % 2 == 0) {
    const int h1 = H1 / 2;
    for (int it = threadIdx.x; it < (H / 2) << lks; it += NT) {
      const int s = it & (KS - 1), rest = it >> lks;  // n2 * h1 + k1, k1 < H1 / 2
      const int n2 = rest / h1, k1 = rest - n2 * h1;
      T2 a, b;
      dft_pair<CONJ, 4>(Fl + k1 * H1, X + (n2 << lks) + s, s1, H1, a, b);
      const int ia = ((n2 * H1 + k1) << lks) + s;
      Y[ia] = post(a, n2 * k1);
      Y[ia + (h1 << lks)] = post(b, n2 * (k1 + h1));
    }
  } else {
    for (int it = threadIdx.x; it < H << lks; it += NT) {
      const int s = it & (KS - 1), rest = it >> lks;  // n2 * H1 + k1
      const int n2 = rest / H1, k1 = rest - n2 * H1;
      Y[it] = post(dft_one<CONJ>(Fl + k1 * H1, X + (n2 << lks) + s, s1, H1), n2 * k1);
    }
  }
}

// Step 2: the H2-point DFTs over n2; emit(k, s, x) receives output
// k = k1 + H1 k2 of site s.
template <typename T, int NT, bool CONJ, class Emit>
FPH_DEVINL void bpc_step2(const typename Cplx<T>::type* F2, const typename Cplx<T>::type* Y, int H1,
                          int H2, int lks, const Emit& emit) {
  using T2 = typename Cplx<T>::type;
  const int KS = 1 << lks, H = H1 * H2, s2 = H1 << lks;
  if (H2 % 2 == 0) {
    for (int it = threadIdx.x; it < (H / 2) << lks; it += NT) {
      const int s = it & (KS - 1), kk = it >> lks;  // k1 + H1 k2, k2 < H2 / 2
      const int k2 = kk / H1, k1 = kk - k2 * H1;
      T2 a, b;
      dft_pair<CONJ, 4>(F2 + k2 * H2, Y + (k1 << lks) + s, s2, H2, a, b);
      emit(kk, s, a);
      emit(kk + H / 2, s, b);
    }
  } else {
    for (int it = threadIdx.x; it < H << lks; it += NT) {
      const int s = it & (KS - 1), kk = it >> lks;
      const int k2 = kk / H1, k1 = kk - k2 * H1;
      emit(kk, s, dft_one<CONJ>(F2 + k2 * H2, Y + (k1 << lks) + s, s2, H2));
    }
  }
}

// The DFT matrices and twiddles into LDS (bpc_lds_tables values).
template <typename T, int NT>
FPH_DEVINL void bpc_tables(const PcView<T>& pc, typename Cplx<T>::type* tab) {
  const int H = pc.H, nF = pc.H1 * pc.H1 + pc.H2 * pc.H2;
  for (int k = threadIdx.x; k < nF; k += NT) tab[k] = pc.F[k];
  for (int k = threadIdx.x; k < H; k += NT) tab[nF + k] = pc.W[k];
}

// Forward transform of r ([Ltau][N]) into Z ([H][N] complex), tables in tab.
template <typename T, int NT, int BUDGET>
FPH_DEVINL void bpc_forward(const Geom& g, const PcView<T>& pc, const T* __restrict__ r,
                            typename Cplx<T>::type* __restrict__ Z, const typename Cplx<T>::type* tab,
                            typename Cplx<T>::type* lds) {
  using T2 = typename Cplx<T>::type;
  const int H = pc.H, H1 = pc.H1, H2 = pc.H2, lks = bpc_tile_log2(g.N, H, BUDGET, sizeof(T2)), KS = 1 << lks;
  const int nF = H1 * H1 + H2 * H2;
  const T2* Fl = tab;
  const T2* Wl = Fl + nF;
  T2* Y0 = lds;
  T2* Y1 = Y0 + (H << lks);
  const T scale = (T)(1.0 / sqrt((double)g.Ltau));
  const long hN = (long)H * g.N;
  for (int i0 = 0; i0 < g.N; i0 += KS) {
    // stage 0: y_tau = e^{-i pi tau/Ltau} (r_tau - i r_{tau+H}); a site past
    // the end of a ragged tile repeats the last one and is not written out
#pragma unroll 4
    for (int e = threadIdx.x; e < H << lks; e += NT) {
      const int tau = e >> lks;
      const long o = (long)tau * g.N + min(i0 + (e & (KS - 1)), g.N - 1);
      const T a = r[o], b = r[o + hN];
      const T2 t = pc.tw[tau];
      Y0[e] = T2{t.x * a + t.y * b, t.y * a - t.x * b};
    }
    __syncthreads();
    bpc_step1<T, NT, false>(Fl, Wl, Y0, Y1, H1, H2, lks);
    __syncthreads();
    bpc_step2<T, NT, false>(Fl + H1 * H1, Y1, H1, H2, lks, [&](int k, int s, T2 x) {
      if (i0 + s < g.N) Z[(long)k * g.N + i0 + s] = T2{x.x * scale, x.y * scale};
    });
    // the next tile's step 1, which rewrites Y1, comes after its own barrier
  }
  __syncthreads();
}

// Inverse transform of Z into z ([Ltau][N]); returns (thread-local)
// partial sums of r . z.
template <typename T, int NT, int BUDGET>
FPH_DEVINL double bpc_inverse(const Geom& g, const PcView<T>& pc,
                              const typename Cplx<T>::type* __restrict__ Z, const T* __restrict__ r,
                              T* __restrict__ z, const typename Cplx<T>::type* tab,
                              typename Cplx<T>::type* lds) {
  using T2 = typename Cplx<T>::type;
  const int H = pc.H, H1 = pc.H1, H2 = pc.H2, lks = bpc_tile_log2(g.N, H, BUDGET, sizeof(T2)), KS = 1 << lks;
  const int nF = H1 * H1 + H2 * H2;
  const T2* Fl = tab;
  const T2* Wl = Fl + nF;
  T2* Zt = lds;
  T2* Y = Zt + (H << lks);
  const T scale = (T)(2.0 / sqrt((double)g.Ltau));
  const long hN = (long)H * g.N;
  double acc_dot = 0.0;
  for (int i0 = 0; i0 < g.N; i0 += KS) {
#pragma unroll 4
    for (int e = threadIdx.x; e < H << lks; e += NT)
      Zt[e] = Z[(long)(e >> lks) * g.N + min(i0 + (e & (KS - 1)), g.N - 1)];
    __syncthreads();
    bpc_step1<T, NT, true>(Fl, Wl, Zt, Y, H1, H2, lks);
    __syncthreads();
    bpc_step2<T, NT, true>(Fl + H1 * H1, Y, H1, H2, lks, [&](int tau, int s, T2 x) {
      if (i0 + s >= g.N) return;
      const T2 sv = cmulc<T2, T>(x, pc.tw[tau]);
      const long oa = (long)tau * g.N + i0 + s;
      const T va = scale * sv.x, vb = -scale * sv.y;
      z[oa] = va;
      z[oa + hN] = vb;
      acc_dot += (double)r[oa] * (double)va + (double)r[oa + hN] * (double)vb;
    });
  }
  __syncthreads();
  return acc_dot;
}

// The coefficients of one block for a wave that runs it alone: lane l holds
// c_l, then c_{64 + l}, ..., and a step takes its own by a lane read (a table
// in memory would put a load's latency into every step).
template <typename T2>
struct WaveCoef {
  const T2* p;
  int NP;
  mutable T2 mine;
  mutable int at;  // first coefficient held
  FPH_DEVINL WaveCoef(const T2* pp, int n) : p(pp), NP(n), at(0) { load(); }
  FPH_DEVINL void load() const { mine = p[min(at + (int)(threadIdx.x & 63), NP - 1)]; }
  FPH_DEVINL T2 operator[](int m) const {
    m = __builtin_amdgcn_readfirstlane(m);
    if ((m & ~63) != at) {
      at = m & ~63;
      load();
    }
    return T2{lane_read(mine.x, m & 63), lane_read(mine.y, m & 63)};
  }
  static FPH_DEVINL double lane_read(double v, int l) { return readlane_d(v, l); }
  static FPH_DEVINL float lane_read(float v, int l) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
  }
};

// The coefficients of one block, zero from its own N_P on: the blocks of a
// round share its longest series' steps.
template <typename T2>
struct BpcCoef {
  const T2* p;
  int NP;
  FPH_DEVINL T2 operator[](int m) const {
    const T2 v = p[min(m, NP - 1)];
    const bool in = m < NP;
    return T2{in ? v.x : 0, in ? v.y : 0};
  }
};

// F F^T on every frequency block of Z, in place: block k gets the
// conjugate series in A^T, then the series in A (as k_kpm with op 2).  Up to
// kBpcWaveQ plaquettes each wave runs blocks of its own, its parts on its two
// halves and without barriers (cheb_series_split), after the longest blocks as
// matrices where there are any.  Else the workgroup takes the blocks in rounds of G, longest series first (order o
// serves frequency w' = o, and N_P does not grow with it), each group of Q
// threads one block in its own LDS buffers, all with the step count of the
// round's first block, so every thread takes the same barriers.  Threads
// without a plaquette or a block run the same branch-free steps on spare LDS
// entries.  The coefficients are read from the table in global memory;
// consecutive series need no barrier between them beyond the one cheb_series
// itself takes.  th = tanh(dtau t) (the primed checkerboard factors).
template <typename T, int NT, int BUDGET>
FPH_DEVINL void bpc_series(const Geom& g, const PcView<T>& pc, T th,
                           typename Cplx<T>::type* __restrict__ Z, typename Cplx<T>::type* lds) {
  using T2 = typename Cplx<T>::type;
  const int H = pc.H, G = bpc_groups(g.L, H, NT, BUDGET, sizeof(T2));
  const int nbuf = 2 * kpm_row_stride(g.hL) * g.L + kWinPad;
  auto freq = [&](int o) { return (o % 2 == 0) ? o / 2 : H - 1 - o / 2; };
  if (g.Q <= kBpcWaveQ) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, q = lane & 31;
    const bool im = lane >= 32, own = q < g.Q;
    const Win w = make_win(g, q, own);
    const int i0 = w.x0 + w.row[1], iL = i0 + g.L;
    const T sA = (T)pc.info->s, cA = (T)pc.info->c;
    const T db[4] = {pc.c4 * pc.dbar[i0], pc.c4 * pc.dbar[i0 + 1], pc.c4 * pc.dbar[iL],
                     pc.c4 * pc.dbar[iL + 1]};
    T* buf0 = reinterpret_cast<T*>(lds) + (4L * min(wave, G - 1) + (im ? 1 : 0)) * nbuf;
    T* buf1 = buf0 + 2 * nbuf;
    auto swap = [&](const T (&v)[4], T (&o)[4]) {
#pragma unroll
      for (int m = 0; m < 4; ++m) o[m] = __shfl_xor(v[m], 32, 64);
    };
    // The longest blocks as matrices, a thread per row, up to 36 sites (L = 4, 6; a
    // row is a chain of loads eight columns at a time, at L = 8 longer than the
    // series: 28 000 against 16 000 cycles at Ltau 32): G is Hermitian, so the lanes
    // read along its rows and take the conjugate.
    // (A workgroup applies them to its one vector: class 0.)
    constexpr int kP = sizeof(T) == 8 ? 0 : 1;
    const int kd = pc.dense == nullptr || g.N > kBpcDenseN ? 0 : min(pc.info->want[kP][0], pc.info->built[kP]);
    for (int o0 = 0, per = NT / g.N; o0 < kd; o0 += per) {
      const int o = o0 + (int)threadIdx.x / g.N, row = threadIdx.x % g.N;
      const bool mine = (int)threadIdx.x < per * g.N && o < kd;
      T2* Zk = Z + (long)freq(mine ? o : o0) * g.N;
      const T2* Gr = pc.dense + (long)(mine ? o : o0) * g.N * g.N + row;
      T2 acc = T2{0, 0};
#pragma unroll 8
      for (int c = 0; c < g.N; ++c) cmacc(acc, Gr[(long)c * g.N], Zk[c]);
      __syncthreads();  // every row of these blocks has read its values
      if (mine) Zk[row] = acc;
    }
    if (wave < G) {
      for (int o = kd + wave; o < H; o += G) {
        const int k = freq(o), NP = __builtin_amdgcn_readfirstlane(pc.np[2 * k]);
        const WaveCoef<T2> cf(pc.coef + (long)k * kNPMax, NP), cft(pc.coef + (long)k * kNPMax, NP);
        T2* Zk = Z + (long)k * g.N;
        T2 z[4];
        ld2c(Zk + i0, z[0], z[1]);
        ld2c(Zk + iL, z[2], z[3]);
        T x[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) x[m] = sel(im, z[m].y, z[m].x);
        cheb_series_split<T, true, false, true>(w, NP, cft, sA, cA, x, db, buf0, buf1, th, im, q, g.Q, swap);
        cheb_series_split<T, false, false, true>(w, NP, cf, sA, cA, x, db, buf0, buf1, th, im, q, g.Q, swap);
        T o4[4];
        swap(x, o4);
        const T t0 = sel(im, o4[2], o4[0]), t1 = sel(im, o4[3], o4[1]);
        if (own)  // row y0 by the real lane, row y0+1 by the imaginary one
          st2c(Zk + (im ? iL : i0), T2{sel(im, t0, x[0]), sel(im, x[2], t0)},
               T2{sel(im, t1, x[1]), sel(im, x[3], t1)});
      }
    }
    __syncthreads();
    return;
  }
  const int grp = min((int)threadIdx.x / g.Q, G);
  const int q = threadIdx.x - grp * g.Q;
  const bool lane_ok = grp < G;
  T2* buf0 = lds + 2L * (lane_ok ? grp : 0) * nbuf;
  T2* buf1 = buf0 + nbuf;
  const Win w = make_win(g, q, lane_ok);
  const int i0 = w.x0 + w.row[1], iL = i0 + g.L;
  const T sA = (T)pc.info->s, cA = (T)pc.info->c;
  const T db[4] = {pc.c4 * pc.dbar[i0], pc.c4 * pc.dbar[i0 + 1], pc.c4 * pc.dbar[iL],
                       pc.c4 * pc.dbar[iL + 1]};
  for (int o0 = 0; o0 < H; o0 += G) {
    const int NP = pc.np[2 * freq(o0)];
    const bool own = lane_ok && o0 + grp < H;
    const int k = freq(own ? o0 + grp : o0);
    T2* Zk = Z + (long)k * g.N;
    T2 x[4], acc[4];
    ld2c(Zk + i0, x[0], x[1]);
    ld2c(Zk + iL, x[2], x[3]);
    const BpcCoef<T2> cf{pc.coef + (long)k * kNPMax, pc.np[2 * k]};
    cheb_series<T, true, false>(w, NP, cf, sA, cA, x, db, buf0, buf1, th, acc, q, g.Q);
#pragma unroll
    for (int m = 0; m < 4; ++m) x[m] = acc[m];
    cheb_series<T, false, false>(w, NP, cf, sA, cA, x, db, buf0, buf1, th, acc, q, g.Q);
    if (own) {
      st2c(Zk + i0, acc[0], acc[1]);
      st2c(Zk + iL, acc[2], acc[3]);
    }
  }
  __syncthreads();
}

}  // namespace fph
