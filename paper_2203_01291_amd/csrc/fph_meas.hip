// Stochastic Green's-function measurements with FFT acceleration (Sec. VI),
// built on the solver's C ABI (fermion_matvec, pcg_solve) plus the discrete
// Fourier transforms of this file.
//
// Grid: vectors are v[tau][i], i = x + L*y; a 3-D transform acts on
// (tau, y, x) as a spatial 2-D transform per time slice (k_fft_xy) and a
// transform along tau per site (k_fft_t).  Both are mixed-radix Stockham
// FFTs in LDS: radices 8, 5, 4, 3 and 2 as register butterflies, larger prime
// factors as direct sums, so 5 n log2 n operations per line instead of the
// n (P + Q) of a two-factor direct form; short sides are direct (k_dft_xy).
//  * Correlations need only the real part of the last inverse transform, and
//    for complex sequences z = a1 + i a2, w = b1 + i b2
//      Re sum_i conj(z_i) w_{i+D} = (a1 * b1)_D + (a2 * b2)_D,
//    so one complex pair (z, w) carries two real pairs, with no untangling:
//    the sums over pairs run over half as many transforms.
//  * The tau pass transforms z and w of the same sites in one workgroup,
//    loops over the pairs of a launch and keeps sum conj(Z) W in registers:
//    transformed grids are never written.
//  * The "twisted" variant multiplies the input by exp(-i pi tau/Ltau) first:
//    it is the transform, on the Ltau odd frequencies, of a sequence extended
//    antiperiodically to 2 Ltau slices, which is how the imaginary-time
//    antiperiodicity of G^ext (Eq. G_def-1) enters; its inverse multiplies
//    the output by exp(+i pi tau/Ltau).
// Transforms are unnormalised (forward exp(-2 pi i k n / n_d), inverse
// exp(+...)); the estimators fold every normalisation into one final scale.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>

#include "../../include/holstein_hmc.h"
#include "fph_common.h"
#include "fph_internal.h"

namespace {

constexpr int kLdsMax = 150 * 1024;  // dynamic LDS budget per workgroup

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cfma(double2 a, double2 b, double2 c) {  // c + a b
  return make_double2(fma(a.x, b.x, fma(-a.y, b.y, c.x)), fma(a.x, b.y, fma(a.y, b.x, c.y)));
}
__device__ __forceinline__ double2 conjd(double2 a) { return make_double2(a.x, -a.y); }

// tw[m] = exp(-2 pi i m / n), m < n, to the last bits: the rounding of 2 m / n,
// which its sine and cosine would carry on, is put right to first order.
__global__ void __launch_bounds__(256) k_meas_twiddles(int n, double2* __restrict__ tw) {
  for (int m = blockIdx.x * 256 + threadIdx.x; m < n; m += gridDim.x * 256) {
    double s, c;
    const double t = 2.0 * m / n, e = M_PI * (fma(-t, (double)n, 2.0 * m) / n);
    sincospi(t, &s, &c);
    tw[m] = make_double2(fma(-s, e, c), -fma(c, e, s));
  }
}

// ------------------------------------------------------------- line FFT

constexpr int kMaxStages = 12;

// Stockham plan of one length: radices (an even one first, so that the first
// stage is a register butterfly) and, per stage, magic numbers that divide by
// the product Ns of the earlier radices and by n / R.
struct FftPlan {
  int n, ns;
  int R[kMaxStages];
  unsigned mNs[kMaxStages], mNb[kMaxStages];
  unsigned mn;
};

// ceil(2^32 / d): e / d = __umulhi(e, m) while e d < 2^32 (here below 2^24);
// 0 stands for d = 1.
unsigned magic(unsigned d) { return d <= 1 ? 0u : (unsigned)(((1ull << 32) + d - 1) / d); }
__device__ __forceinline__ int udiv(int e, unsigned m) { return m ? (int)__umulhi((unsigned)e, m) : e; }

// small_first: a 4 before the 8s (a first stage from memory has more, smaller butterflies).
FftPlan make_plan(int n, bool small_first) {
  FftPlan p;
  std::memset(&p, 0, sizeof(p));
  p.n = n;
  p.mn = magic(n);
  int twos = 0, m = n;
  while (m % 2 == 0) {
    m /= 2;
    ++twos;
  }
  auto add = [&](int r) { p.R[p.ns++] = r; };
  if (small_first && twos >= 5 && twos % 3 != 0) {
    add(4);
    twos -= 2;
  }
  while (twos >= 5 || twos == 3) {  // 16 is 4 * 4, not 8 * 2
    add(8);
    twos -= 3;
  }
  while (twos >= 2) {
    add(4);
    twos -= 2;
  }
  if (twos) add(2);
  for (int r : {5, 3})
    while (m % r == 0) {
      add(r);
      m /= r;
    }
  for (int r = 7; m > 1; r += 2)
    while (m % r == 0) {
      add(r);
      m /= r;
    }
  int Ns = 1;
  for (int i = 0; i < p.ns; ++i) {
    p.mNs[i] = magic(Ns);
    p.mNb[i] = magic(n / p.R[i]);
    Ns *= p.R[i];
  }
  return p;
}

template <bool INV>
__device__ __forceinline__ double2 mul_i(double2 a) {  // a times -i (forward) or +i
  return INV ? make_double2(-a.y, a.x) : make_double2(a.y, -a.x);
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }

template <bool INV>
__device__ __forceinline__ void dft4(double2& v0, double2& v1, double2& v2, double2& v3) {
  const double2 a = cadd(v0, v2), b = csub(v0, v2), c = cadd(v1, v3), d = mul_i<INV>(csub(v1, v3));
  v0 = cadd(a, c);
  v1 = cadd(b, d);
  v2 = csub(a, c);
  v3 = csub(b, d);
}

// In-place DFT of R values, R in {2, 3, 4, 5, 8}.
template <int R, bool INV>
__device__ __forceinline__ void dft(double2 (&v)[R]) {
  if constexpr (R == 2) {
    const double2 a = v[0];
    v[0] = cadd(a, v[1]);
    v[1] = csub(a, v[1]);
  } else if constexpr (R == 3) {
    constexpr double kS = 0.86602540378443864676;  // sin(2 pi / 3)
    const double2 t = cadd(v[1], v[2]), d = csub(v[1], v[2]);
    const double2 m = make_double2(fma(-0.5, t.x, v[0].x), fma(-0.5, t.y, v[0].y));
    const double2 q = mul_i<INV>(make_double2(kS * d.x, kS * d.y));
    v[0] = cadd(v[0], t);
    v[1] = cadd(m, q);
    v[2] = csub(m, q);
  } else if constexpr (R == 4) {
    dft4<INV>(v[0], v[1], v[2], v[3]);
  } else if constexpr (R == 5) {
    constexpr double c1 = 0.30901699437494742410, c2 = -0.80901699437494742410;  // cos(2 pi k / 5)
    constexpr double s1 = 0.95105651629515357212, s2 = 0.58778525229247312917;   // sin(2 pi k / 5)
    const double2 t1 = cadd(v[1], v[4]), d1 = csub(v[1], v[4]);
    const double2 t2 = cadd(v[2], v[3]), d2 = csub(v[2], v[3]);
    const double2 m1 = make_double2(fma(c2, t2.x, fma(c1, t1.x, v[0].x)), fma(c2, t2.y, fma(c1, t1.y, v[0].y)));
    const double2 m2 = make_double2(fma(c1, t2.x, fma(c2, t1.x, v[0].x)), fma(c1, t2.y, fma(c2, t1.y, v[0].y)));
    const double2 q1 = mul_i<INV>(make_double2(fma(s2, d2.x, s1 * d1.x), fma(s2, d2.y, s1 * d1.y)));
    const double2 q2 = mul_i<INV>(make_double2(fma(-s1, d2.x, s2 * d1.x), fma(-s1, d2.y, s2 * d1.y)));
    v[0] = cadd(v[0], cadd(t1, t2));
    v[1] = cadd(m1, q1);
    v[4] = csub(m1, q1);
    v[2] = cadd(m2, q2);
    v[3] = csub(m2, q2);
  } else {
    static_assert(R == 8, "radix");
    constexpr double kH = 0.70710678118654752440;
    dft4<INV>(v[0], v[2], v[4], v[6]);
    dft4<INV>(v[1], v[3], v[5], v[7]);
    const double2 i3 = mul_i<INV>(v[3]), i7 = mul_i<INV>(v[7]);
    const double2 o1 = make_double2(kH * (v[3].x + i3.x), kH * (v[3].y + i3.y));
    const double2 o2 = mul_i<INV>(v[5]);
    const double2 o3 = make_double2(kH * (i7.x - v[7].x), kH * (i7.y - v[7].y));
    const double2 e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6], o0 = v[1];
    v[0] = cadd(e0, o0);
    v[4] = csub(e0, o0);
    v[1] = cadd(e1, o1);
    v[5] = csub(e1, o1);
    v[2] = cadd(e2, o2);
    v[6] = csub(e2, o2);
    v[3] = cadd(e3, o3);
    v[7] = csub(e3, o3);
  }
}

// One Stockham stage of radix R over `items` = (n / R) lines' butterflies:
// split(e, s, j) gives item e's line s and butterfly j; ld(i, s) and
// st(i, s, v) read and write entry i of line s; tw[m] = w_n^m (conjugated for
// INV).  Butterfly j, k = j mod Ns: inputs j + r n/R times w^{k r n/(Ns R)},
// outputs (j - k) R + k + r Ns.
template <int R, bool INV, int NT, class Split, class Ld, class St>
__device__ __forceinline__ void fft_stage(int n, int Ns, unsigned mNs, int items, const double2* tw,
                                          const Split& split, const Ld& ld, const St& st) {
  const int nb = n / R, ts = nb / Ns;
  for (int e = threadIdx.x; e < items; e += NT) {
    int s, j;
    split(e, s, j);
    const int k = j - udiv(j, mNs) * Ns;
    double2 v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = ld(j + r * nb, s);
    if (Ns > 1) {
#pragma unroll
      for (int r = 1; r < R; ++r) v[r] = cmul(v[r], tw[k * r * ts]);
    }
    dft<R, INV>(v);
    const int o = (j - k) * R + k;
#pragma unroll
    for (int r = 0; r < R; ++r) st(o + r * Ns, s, v[r]);
  }
}

// The same for any radix, one output at a time by its direct sum (prime
// factors above 5).
template <int NT, class Split, class Ld, class St>
__device__ __forceinline__ void fft_stage_any(int R, int n, int Ns, unsigned mNs, int items, const double2* tw,
                                              const Split& split, const Ld& ld, const St& st) {
  const int nb = n / R, ts = nb / Ns;
  for (int e = threadIdx.x; e < items * R; e += NT) {
    const int r = e / items;
    int s, j;
    split(e - r * items, s, j);
    const int k = j - udiv(j, mNs) * Ns;
    const int step = k * ts + r * nb;  // (below n)
    double2 acc = make_double2(0.0, 0.0);
    int m = 0;
#pragma unroll 4
    for (int q = 0; q < R; ++q) {
      acc = cfma(ld(j + q * nb, s), tw[m], acc);
      m += step;
      if (m >= n) m -= n;
    }
    st((j - k) * R + k + r * Ns, s, acc);
  }
}

template <bool INV, int NT, class Split, class Ld, class St>
__device__ __forceinline__ void fft_stage_sel(int R, int n, int Ns, unsigned mNs, int items, const double2* tw,
                                              const Split& split, const Ld& ld, const St& st) {
  switch (R) {
    case 8: fft_stage<8, INV, NT>(n, Ns, mNs, items, tw, split, ld, st); break;
    case 5: fft_stage<5, INV, NT>(n, Ns, mNs, items, tw, split, ld, st); break;
    case 4: fft_stage<4, INV, NT>(n, Ns, mNs, items, tw, split, ld, st); break;
    case 3: fft_stage<3, INV, NT>(n, Ns, mNs, items, tw, split, ld, st); break;
    case 2: fft_stage<2, INV, NT>(n, Ns, mNs, items, tw, split, ld, st); break;
    default: fft_stage_any<NT>(R, n, Ns, mNs, items, tw, split, ld, st); break;
  }
}

// The first stage of a line of even length (make_plan starts with 8, 4 or 2): its
// loads from memory sit in a stage of their own, one kind of load per instance,
// so that a butterfly issues all of them before it waits for the first.
template <bool INV, int NT, class Split, class Ld, class St>
__device__ __forceinline__ void fft_first(int R, int n, int items, const Split& split, const Ld& ld, const St& st) {
  switch (R) {
    case 8: fft_stage<8, INV, NT>(n, 1, 0u, items, nullptr, split, ld, st); break;
    case 4: fft_stage<4, INV, NT>(n, 1, 0u, items, nullptr, split, ld, st); break;
    default: fft_stage<2, INV, NT>(n, 1, 0u, items, nullptr, split, ld, st); break;
  }
}

// ------------------------------------------------------------ space pass

// One grid of a space launch.  Input: complex `in`, or a b + i c d of real
// vectors (b or d null: that factor is 1; c null: no imaginary part).
// Output: complex `out`, or the real part times `scale` in `outr`.
struct XyJob {
  const double2* in;
  const double *a, *b, *c, *d;
  double2* out;
  double* outr;
};
constexpr int kGrids = 8;  // grids per launch, and complex grids of workspace
struct XyArgs {
  XyJob job[kGrids];
  int njob;
  double scale;
};

// Spatial transform, one workgroup per (time slice, grid).  Stages along y
// first (lanes along x: the first stage reads rows from memory straight into
// its butterflies), then along x (the last stage writes rows from its
// butterflies, lanes along its contiguous outputs).  LDS rows are L + 1 long,
// odd, so that lanes along y do not meet on a bank.  The grids of a slice are
// numbered next to each other on one XCD: they read the same vectors.
// Bound by its traffic from the caches (reads of up to four real vectors and
// one complex write per grid) and the chain of stages: 43 us for eight grids
// of 400 x 32 x 32, 14-15 us each with direct DFTs and one grid per launch; with
// the 4 before the 8s along y the ten-vector estimators took 1.16 ms, 1.25 before.
template <bool INV, int NT>
__global__ void __launch_bounds__(NT)
k_fft_xy(int L, int N, FftPlan py, FftPlan px, XyArgs A, const double2* __restrict__ twL) {
  extern __shared__ double2 sh[];
  const int LP = L + 1;
  double2* tw = sh;
  double2* buf = sh + L;
  const int nbuf = L * LP;
  const int logical = fph::xcd_contiguous(blockIdx.x, gridDim.x);
  const int slice = logical / A.njob;
  const XyJob jb = A.job[logical - slice * A.njob];
  const long base = (long)slice * N;
  for (int e = threadIdx.x; e < L; e += NT) tw[e] = INV ? conjd(twL[e]) : twL[e];
  auto lanes_x = [&](int e, int& s, int& j) {
    j = udiv(e, px.mn);
    s = e - j * L;
  };
  {  // along y, from memory: row y = k, column x = s
    const int R = py.R[0], items = L / R * L;
    auto st = [&](int k, int s, double2 v) { buf[nbuf + k * LP + s] = v; };
    auto at = [&](int k, int s) { return base + (long)k * L + s; };
    auto first = [&](const auto& ld) {
      fft_first<INV, NT>(R, L, items, lanes_x, [&](int k, int s) { return ld(at(k, s)); }, st);
    };
    if (jb.in) first([&](long o) { return jb.in[o]; });
    else if (jb.b && jb.c) first([&](long o) { return make_double2(jb.a[o] * jb.b[o], jb.c[o] * jb.d[o]); });
    else if (jb.b) first([&](long o) { return make_double2(jb.a[o] * jb.b[o], 0.0); });
    else if (jb.c) first([&](long o) { return make_double2(jb.a[o], jb.c[o]); });
    else first([&](long o) { return make_double2(jb.a[o], 0.0); });
  }
  int cur = 1, Ns = py.R[0];
  for (int t = 1; t < py.ns + px.ns - 1; ++t) {  // along y, then along x
    const bool x = t >= py.ns;
    const int i = x ? t - py.ns : t, sn = x ? 1 : LP, sb = x ? LP : 1;
    const int R = x ? px.R[i] : py.R[i];
    if (i == 0) Ns = 1;
    const double2* src = buf + cur * nbuf;
    double2* dst = buf + (cur ^ 1) * nbuf;
    __syncthreads();
    fft_stage_sel<INV, NT>(
        R, L, Ns, x ? px.mNs[i] : py.mNs[i], L / R * L, tw, lanes_x,
        [&](int k, int s) { return src[k * sn + s * sb]; }, [&](int k, int s, double2 v) { dst[k * sn + s * sb] = v; });
    Ns *= R;
    cur ^= 1;
  }
  {  // the last along x, to memory: row y = s, column x = k, lanes along its outputs
    const int i = px.ns - 1, R = px.R[i], nb = L / R;
    if (i == 0) Ns = 1;
    const double2* src = buf + cur * nbuf;
    auto split = [&](int e, int& s, int& j) {
      s = udiv(e, px.mNb[i]);
      j = e - s * nb;
    };
    auto ld = [&](int k, int s) { return src[k + s * LP]; };
    auto last = [&](const auto& put) {
      fft_stage_sel<INV, NT>(R, L, Ns, px.mNs[i], nb * L, tw, split, ld,
                             [&](int k, int s, double2 v) { put(base + (long)s * L + k, v); });
    };
    __syncthreads();
    if (jb.outr) last([&](long o, double2 v) { jb.outr[o] = A.scale * v.x; });
    else last([&](long o, double2 v) { jb.out[o] = v; });
  }
}

// The same by direct DFTs of length L in three phases, for short sides (the rule
// stands with launch_xy).  A small transform is a chain of phases (a barrier, an
// LDS round trip, the fetch of the stage's instructions: 0.5 to 0.8 us), and a
// side of 2 p is two stages per axis with a direct sum over p in it anyway.  One
// grid of 40 slices, L = 6 and 22: 3.6 and 5.2 us; as FFTs 5.6 and 7.9.
template <bool INV, int NT>
__global__ void __launch_bounds__(NT)
k_dft_xy(int L, int N, XyArgs A, const double2* __restrict__ twL) {
  extern __shared__ double2 sh[];
  double2* tw = sh;
  double2* U = sh + L;  // [y][x]
  double2* B = U + N;   // [y][kx]
  const int slice = blockIdx.x / A.njob;
  const XyJob jb = A.job[blockIdx.x - slice * A.njob];
  const long base = (long)slice * N;
  for (int e = threadIdx.x; e < L; e += NT) tw[e] = INV ? conjd(twL[e]) : twL[e];
  auto fill = [&](const auto& ld) {
    for (int e = threadIdx.x; e < N; e += NT) U[e] = ld(base + e);
  };
  if (jb.in) fill([&](long o) { return jb.in[o]; });
  else if (jb.b) fill([&](long o) { return make_double2(jb.a[o] * jb.b[o], jb.c ? jb.c[o] * jb.d[o] : 0.0); });
  else fill([&](long o) { return make_double2(jb.a[o], jb.c ? jb.c[o] : 0.0); });
  __syncthreads();
  // Entries x and L - x of a line meet outputs k and L - k with the same cosine
  // and sine (w = c + i t): with p, q their sum and difference,
  // X_k, X_{L-k} = v_0 + (-1)^k v_{L/2} + sum c p +- i sum t q, odd and even x
  // summed apart (a shorter chain, and as small an error as the FFT's).
  const int h = L / 2;
  auto pair = [&](const double2* v, int stride, int k, double2& lo, double2& hi) {
    double2 C[2], S[2];
    C[0] = C[1] = S[0] = S[1] = make_double2(0.0, 0.0);
    int m = 0;
    for (int x = 1; x < h; x += 2) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        if (x + i == h) break;
        m += k;
        if (m >= L) m -= L;
        const double2 w = tw[m], f = v[(x + i) * stride], g = v[(L - x - i) * stride];
        const double2 p = cadd(f, g), q = csub(f, g);
        C[i] = make_double2(fma(w.x, p.x, C[i].x), fma(w.x, p.y, C[i].y));
        S[i] = make_double2(fma(w.y, q.x, S[i].x), fma(w.y, q.y, S[i].y));
      }
    }
    const double2 v0 = v[0], vh = v[h * stride];
    const double2 c = cadd(k & 1 ? csub(v0, vh) : cadd(v0, vh), cadd(C[0], C[1])), t = cadd(S[0], S[1]);
    lo = make_double2(c.x - t.y, c.y + t.x);
    hi = make_double2(c.x + t.y, c.y - t.x);
  };
  for (int e = threadIdx.x; e < (h + 1) * L; e += NT) {  // along x
    const int y = e / (h + 1), k = e - y * (h + 1);
    double2 lo, hi;
    pair(U + y * L, 1, k, lo, hi);
    B[y * L + k] = lo;
    if (k > 0) B[y * L + L - k] = hi;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < (h + 1) * L; e += NT) {  // along y
    const int ky = e / L, k = e - ky * L;
    double2 lo, hi;
    pair(B + k, L, ky, lo, hi);
    const long o = base + (long)ky * L + k, o2 = base + (long)(L - ky) * L + k;
    if (jb.outr) {
      jb.outr[o] = A.scale * lo.x;
      if (ky > 0) jb.outr[o2] = A.scale * hi.x;
    } else {
      jb.out[o] = lo;
      if (ky > 0) jb.out[o2] = hi;
    }
  }
}

// ------------------------------------------------------------- time pass

enum { T_PLAIN = 0, T_CROSS = 1, T_PREFIX = 2 };
constexpr int kTNT = 512;          // threads of a time workgroup
constexpr int kTElems = 2048;      // its most elements, T * S
constexpr int kTE = kTElems / kTNT;

// T_PLAIN: out[0] = transform of z[0][0].  T_CROSS, set y = blockIdx.y: out[y]
// += sum_p conj(Z_p) W_p, p < np.  T_PREFIX: for p < np in order out[0] +=
// conj(run) Z_p, run += Z_p.  first: out and run start from zero.
struct TArgs {
  const double2* z[2][kGrids];
  const double2* w[2][kGrids];
  double2* out[2];
  double2* run;
  int np, first, twist;
};

// Transform along tau of S = 2^ls sites per workgroup (grid: N/S tiles, sets).
// tw2[m] = exp(-i pi m / T), m < 2T.  The first stage reads its inputs from
// memory; the sums over pairs stay in registers, one element per thread and
// step of kTNT.  Eight grids of 400 x 32 x 32 with their products: 29 us; the
// two-factor direct form took 17 us per grid and 5 us per product pass.
template <bool INV, int MODE>
__global__ void __launch_bounds__(kTNT)
k_fft_t(int N, int ls, FftPlan pl, TArgs A, const double2* __restrict__ tw2) {
  extern __shared__ double2 sh[];
  const int T = pl.n, S = 1 << ls, nel = T << ls;
  double2* tw = sh;
  double2* buf = sh + T;
  const int set = blockIdx.y;
  const int site0 = fph::xcd_contiguous(blockIdx.x, gridDim.x) << ls;
  for (int e = threadIdx.x; e < T; e += kTNT) tw[e] = INV ? conjd(tw2[2 * e]) : tw2[2 * e];
  __syncthreads();
  auto split = [&](int e, int& s, int& j) {
    s = e & (S - 1);
    j = e >> ls;
  };
  // Transform of `in`; returns the buffer that holds it ([tau][s]), after a barrier.
  auto transform = [&](const double2* in) {
    int cur = 1, Ns = pl.R[0];
    {
      const int items = (T / Ns) << ls;
      auto put = [&](int k, int s, double2 v) { buf[nel + (k << ls) + s] = v; };
      auto get = [&](int k, int s) { return in[(long)k * N + site0 + s]; };
      if (!INV && A.twist)
        fft_first<INV, kTNT>(Ns, T, items, split, [&](int k, int s) { return cmul(get(k, s), tw2[k]); }, put);
      else
        fft_first<INV, kTNT>(Ns, T, items, split, get, put);
      __syncthreads();
    }
    for (int i = 1; i < pl.ns; ++i) {
      const int R = pl.R[i];
      const double2* src = buf + cur * nel;
      double2* dst = buf + (cur ^ 1) * nel;
      auto ld = [&](int k, int s) { return src[(k << ls) + s]; };
      auto st = [&](int k, int s, double2 v) { dst[(k << ls) + s] = v; };
      fft_stage_sel<INV, kTNT>(R, T, Ns, pl.mNs[i], (T / R) << ls, tw, split, ld, st);
      __syncthreads();
      Ns *= R;
      cur ^= 1;
    }
    return (const double2*)(buf + cur * nel);
  };
  auto at = [&](int e) { return (long)(e >> ls) * N + site0 + (e & (S - 1)); };
  if constexpr (MODE == T_PLAIN) {
    const double2* x = transform(A.z[0][0]);
    for (int e = threadIdx.x; e < nel; e += kTNT) {
      double2 v = x[e];
      if (INV && A.twist) v = cmul(v, conjd(tw2[e >> ls]));
      A.out[0][at(e)] = v;
    }
  } else {
    double2 acc[kTE], keep[kTE];  // keep: Z_p (T_CROSS) or the running sum (T_PREFIX)
    double2* out = A.out[set];
#pragma unroll
    for (int i = 0; i < kTE; ++i) {
      const int e = threadIdx.x + i * kTNT;
      acc[i] = keep[i] = make_double2(0.0, 0.0);
      if (e < nel && !A.first) {
        acc[i] = out[at(e)];
        if (MODE == T_PREFIX) keep[i] = A.run[at(e)];
      }
    }
    for (int p = 0; p < A.np; ++p) {
      const double2* x = transform(A.z[set][p]);
      if constexpr (MODE == T_CROSS) {
#pragma unroll
        for (int i = 0; i < kTE; ++i) keep[i] = x[min((int)threadIdx.x + i * kTNT, nel - 1)];
        __syncthreads();
        x = transform(A.w[set][p]);
      }
#pragma unroll
      for (int i = 0; i < kTE; ++i) {
        const double2 v = x[min((int)threadIdx.x + i * kTNT, nel - 1)];
        acc[i] = cfma(conjd(keep[i]), v, acc[i]);
        if constexpr (MODE == T_PREFIX) keep[i] = cadd(keep[i], v);
      }
      __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < kTE; ++i) {
      const int e = threadIdx.x + i * kTNT;
      if (e < nel) {
        out[at(e)] = acc[i];
        if (MODE == T_PREFIX) A.run[at(e)] = keep[i];
      }
    }
  }
}

// Whether Ltau = P*Q with P, Q <= 64 (the range of lattices this file takes).
bool slices_ok(int T) {
  for (int p = 1; p <= 64; ++p)
    if (T % p == 0 && T / p <= 64) return T <= kTElems;
  return false;
}

}  // namespace

struct fph_meas_s {
  fph_handle_t h;
  fph_lattice_t lat;
  int max_rhs;
  int L, N, T, ls;
  long d;
  FftPlan pY, pX, pT;
  double2 *twL, *tw2;  // exp(-2 pi i m / L), exp(-i pi m / Ltau)
  double2* grid[kGrids];  // complex grids [Ltau][N]
  double2 *acc, *acc2, *run;
  double* bvec;           // max_rhs real vectors
  size_t lds_xy, lds_t;
};

namespace {

// Threads of a space workgroup: one radix-4 or two radix-8 butterflies each.
hipError_t launch_xy(const fph_meas_s* m, bool inv, const XyArgs& A, hipStream_t s) {
  const dim3 g(m->T * A.njob);
  // Direct sides: up to 22, and up to 38 where a prime factor above 5 is a stage of
  // direct sums (us, direct / FFT, one grid of 40 and of 400 slices: L = 12 4.0 / 5.7
  // and 4.5 / 5.6; 22 5.2 / 7.9 and 6.9 / 10.0; 38 10.5 / 13.5 and 16.7 / 23.3; but 24
  // 5.4 / 5.9 and 7.5 / 7.3, eight grids of 400 18 / 17; 32 8.6 / 6.4 and 14.5 / 9.9).
  // 512 threads where 256 would take the lines in two rounds.
  if (m->L <= 22 || (m->L <= 38 && m->pX.R[m->pX.ns - 1] > 5)) {
    const int nt = (m->L / 2 + 1) * m->L <= 256 ? 256 : 512;
    auto k = nt == 256 ? (inv ? k_dft_xy<true, 256> : k_dft_xy<false, 256>)
                       : (inv ? k_dft_xy<true, 512> : k_dft_xy<false, 512>);
    hipLaunchKernelGGL(k, g, dim3(nt), m->lds_xy, s, m->L, m->N, A, (const double2*)m->twL);
  } else if (m->N <= 1024) {
    auto k = inv ? k_fft_xy<true, 256> : k_fft_xy<false, 256>;
    hipLaunchKernelGGL(k, g, dim3(256), m->lds_xy, s, m->L, m->N, m->pY, m->pX, A, (const double2*)m->twL);
  } else {
    auto k = inv ? k_fft_xy<true, 512> : k_fft_xy<false, 512>;
    hipLaunchKernelGGL(k, g, dim3(512), m->lds_xy, s, m->L, m->N, m->pY, m->pX, A, (const double2*)m->twL);
  }
  return hipGetLastError();
}

template <bool INV, int MODE>
hipError_t launch_t(const fph_meas_s* m, int sets, const TArgs& A, hipStream_t s) {
  hipLaunchKernelGGL((k_fft_t<INV, MODE>), dim3(m->N >> m->ls, sets), dim3(kTNT), m->lds_t, s, m->N, m->ls,
                     m->pT, A, (const double2*)m->tw2);
  return hipGetLastError();
}

TArgs plain_t(const double2* in, double2* out, int twist) {
  TArgs A;
  std::memset(&A, 0, sizeof(A));
  A.z[0][0] = in;
  A.out[0] = out;
  A.twist = twist;
  return A;
}

XyArgs one_xy(const XyJob& j, double scale) {
  XyArgs A;
  std::memset(&A, 0, sizeof(A));
  A.job[0] = j;
  A.njob = 1;
  A.scale = scale;
  return A;
}

// Inverse 3-D transform of `in` (complex), real part times `scale` into out_r.
hipError_t inv3(const fph_meas_s* m, const double2* in, int twist, double scale, double* out_r,
                hipStream_t s) {
  hipError_t e = launch_t<true, T_PLAIN>(m, 1, plain_t(in, m->grid[0], twist), s);
  if (e != hipSuccess) return e;
  return launch_xy(m, true, one_xy(XyJob{m->grid[0], nullptr, nullptr, nullptr, nullptr, nullptr, out_r}, scale),
                   s);
}

}  // namespace

#define MEAS_CHECK(call)                                      \
  do {                                                        \
    hipError_t e_ = (call);                                   \
    if (e_ != hipSuccess) return fph::record_hip_error(e_);   \
  } while (0)

#define MEAS_CALL(call)                \
  do {                                 \
    int rc_ = (call);                  \
    if (rc_ != FPH_OK) return rc_;     \
  } while (0)

extern "C" {

int fph_meas_destroy(fph_meas_t m) {
  if (m == nullptr) return FPH_E_NULL;
  (void)hipDeviceSynchronize();
  void* ptrs[] = {m->twL, m->tw2, m->grid[0], m->acc, m->acc2, m->run, m->bvec};
  for (void* p : ptrs)
    if (p) (void)hipFree(p);
  delete m;
  return FPH_OK;
}

int fph_meas_create(fph_meas_t* out, fph_handle_t h, void* stream) {
  if (out == nullptr || h == nullptr) return FPH_E_NULL;
  *out = nullptr;
  fph_lattice_t lat;
  int32_t max_rhs = 0;
  MEAS_CALL(fph_get_lattice(h, &lat, &max_rhs));
  if (!slices_ok(lat.Ltau)) return FPH_E_LATTICE;
  const int N = lat.L * lat.L;
  const size_t lds_xy = (size_t)(2 * lat.L * (lat.L + 1) + lat.L) * sizeof(double2);
  if (lds_xy > (size_t)kLdsMax) return FPH_E_LATTICE;
  // Sites per time workgroup: a power of two dividing N, at most 8 and kTElems
  // elements, narrower while that leaves fewer than 256 tiles (not below 2).
  int ls = 3;
  while (ls > 0 && ((lat.Ltau << ls) > kTElems || N % (1 << ls) || (ls > 1 && (N >> ls) < 256))) --ls;
  const size_t lds_t = (size_t)(2 * (lat.Ltau << ls) + lat.Ltau) * sizeof(double2);
  if (lds_t > (size_t)kLdsMax) return FPH_E_LATTICE;
  fph_meas_s* m = new fph_meas_s();
  std::memset(m, 0, sizeof(*m));
  m->h = h;
  m->lat = lat;
  m->max_rhs = max_rhs;
  m->L = lat.L;
  m->N = N;
  m->T = lat.Ltau;
  m->ls = ls;
  m->d = (long)N * lat.Ltau;
  m->pY = make_plan(lat.L, true);
  m->pX = make_plan(lat.L, false);
  m->pT = make_plan(lat.Ltau, true);
  m->lds_xy = lds_xy;
  m->lds_t = lds_t;
  hipError_t e = hipSuccess;
#define ALLOC(ptr, bytes) \
  if (e == hipSuccess) e = hipMalloc((void**)&(ptr), (bytes));
  ALLOC(m->twL, m->L * sizeof(double2));
  ALLOC(m->tw2, 2 * m->T * sizeof(double2));
  ALLOC(m->grid[0], kGrids * m->d * sizeof(double2));
  for (int k = 1; k < kGrids; ++k) m->grid[k] = m->grid[0] + k * m->d;
  ALLOC(m->acc, m->d * sizeof(double2));
  ALLOC(m->acc2, m->d * sizeof(double2));
  ALLOC(m->run, m->d * sizeof(double2));
  ALLOC(m->bvec, (size_t)max_rhs * m->d * sizeof(double));
#undef ALLOC
  {
    const void* fns[] = {(const void*)k_fft_xy<false, 256>,    (const void*)k_fft_xy<true, 256>,
                         (const void*)k_fft_xy<false, 512>,    (const void*)k_fft_xy<true, 512>,
                         (const void*)k_dft_xy<false, 256>,    (const void*)k_dft_xy<true, 256>,
                         (const void*)k_dft_xy<false, 512>,    (const void*)k_dft_xy<true, 512>,
                         (const void*)k_fft_t<false, T_PLAIN>, (const void*)k_fft_t<true, T_PLAIN>,
                         (const void*)k_fft_t<false, T_CROSS>, (const void*)k_fft_t<false, T_PREFIX>};
    for (const void* f : fns)
      if (e == hipSuccess) e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsMax);
  }
  hipStream_t s = (hipStream_t)stream;
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_meas_twiddles, dim3(1), dim3(256), 0, s, m->L, m->twL);
    e = hipGetLastError();
  }
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_meas_twiddles, dim3((2 * m->T + 255) / 256), dim3(256), 0, s, 2 * m->T, m->tw2);
    e = hipGetLastError();
  }
  if (e != hipSuccess) {
    fph_meas_destroy(m);
    return fph::record_hip_error(e);
  }
  *out = m;
  return FPH_OK;
}

int meas_fft(fph_meas_t m, int32_t inverse, int32_t twist, const double* in_dev, double* out_dev,
             void* stream) {
  if (m == nullptr || in_dev == nullptr || out_dev == nullptr) return FPH_E_NULL;
  if (in_dev == out_dev) return FPH_E_ARG;
  hipStream_t s = (hipStream_t)stream;
  const double2* in = (const double2*)in_dev;
  double2* out = (double2*)out_dev;
  const int tw = twist != 0;
  const XyJob job{inverse ? m->grid[0] : in, nullptr, nullptr, nullptr, nullptr, inverse ? out : m->grid[0],
                  nullptr};
  if (!inverse) {
    MEAS_CHECK(launch_xy(m, false, one_xy(job, 0.0), s));
    MEAS_CHECK((launch_t<false, T_PLAIN>(m, 1, plain_t(m->grid[0], out, tw), s)));
  } else {
    MEAS_CHECK((launch_t<true, T_PLAIN>(m, 1, plain_t(in, m->grid[0], tw), s)));
    MEAS_CHECK(launch_xy(m, true, one_xy(job, 0.0), s));
  }
  return FPH_OK;
}

int green_vectors(fph_meas_t m, int32_t nvec, const double* xi_dev, double* gxi_dev,
                  const fph_pcg_opts_t* opts, fph_pcg_stats_t* stats_host, void* stream) {
  if (m == nullptr || xi_dev == nullptr || gxi_dev == nullptr || opts == nullptr) return FPH_E_NULL;
  if (nvec < 1) return FPH_E_NRHS;
  fph_pcg_opts_t oo = *opts;
  oo.zero_guess = 1;
  for (int r0 = 0; r0 < nvec; r0 += m->max_rhs) {
    const int nr = (nvec - r0 < m->max_rhs) ? nvec - r0 : m->max_rhs;
    MEAS_CALL(fermion_matvec(m->h, FPH_OP_MT, FPH_F64, nr, xi_dev + (long)r0 * m->d, m->bvec, stream));
    MEAS_CALL(pcg_solve_sync(m->h, nr, m->bvec, gxi_dev + (long)r0 * m->d, &oo,
                        stats_host ? stats_host + r0 : nullptr, stream));
  }
  return FPH_OK;
}

int green_average(fph_meas_t m, int32_t nvec, const double* xi_dev, const double* gxi_dev,
                  double* out_dev, void* stream) {
  if (m == nullptr || xi_dev == nullptr || gxi_dev == nullptr || out_dev == nullptr) return FPH_E_NULL;
  if (nvec < 1) return FPH_E_NRHS;
  hipStream_t s = (hipStream_t)stream;
  // Two vectors per complex pair, kGrids / 2 pairs per launch.
  const long d = m->d;
  for (int n = 0; n < nvec;) {
    XyArgs X;
    TArgs A;
    std::memset(&X, 0, sizeof(X));
    std::memset(&A, 0, sizeof(A));
    A.first = n == 0;
    A.twist = 1;
    A.out[0] = m->acc;
    for (; n < nvec && A.np < kGrids / 2; n += 2, ++A.np) {
      const bool two = n + 1 < nvec;
      for (int k = 0; k < 2; ++k) {
        const double* v = (k ? gxi_dev : xi_dev) + (long)n * d;
        double2* g = m->grid[X.njob];
        X.job[X.njob++] = XyJob{nullptr, v, nullptr, two ? v + d : nullptr, nullptr, g, nullptr};
        (k ? A.w : A.z)[0][A.np] = g;
      }
    }
    MEAS_CHECK(launch_xy(m, false, X, s));
    MEAS_CHECK((launch_t<false, T_CROSS>(m, 1, A, s)));
  }
  // GA = e^{i pi dtau/Ltau} IDFT3[sum_n conj(A_n) B_n] / (nvec Ncal^2), Ncal = N Ltau
  const double ncal = (double)m->d;
  MEAS_CHECK(inv3(m, m->acc, 1, 1.0 / ((double)nvec * ncal * ncal), out_dev, s));
  return FPH_OK;
}

int green_pair_products(fph_meas_t m, int32_t nvec, const double* xi_dev, const double* gxi_dev,
                        double* out_dev, void* stream) {
  if (m == nullptr || xi_dev == nullptr || gxi_dev == nullptr || out_dev == nullptr) return FPH_E_NULL;
  if (nvec < 2) return FPH_E_NRHS;
  hipStream_t s = (hipStream_t)stream;
  const long d = m->d;
  auto xi = [&](int n) { return xi_dev + (long)n * d; };
  auto gx = [&](int n) { return gxi_dev + (long)n * d; };
  const double npairs = 0.5 * (double)nvec * (double)(nvec - 1);
  const double scale = 1.0 / (npairs * (double)d * (double)d);
  // T1: (xi_n . xi_m) * (Gxi_n . Gxi_m);  T3: (xi_n . Gxi_m) * (xi_m . Gxi_n)
  // Two vector pairs per complex pair; kGrids / 4 complex pairs of each
  // product per launch.
  const long npair = (long)nvec * (nvec - 1) / 2;
  int a = 0, b = 1;
  for (long done = 0; done < npair;) {
    XyArgs X;
    TArgs A;
    std::memset(&X, 0, sizeof(X));
    std::memset(&A, 0, sizeof(A));
    A.first = done == 0;
    A.out[0] = m->acc;
    A.out[1] = m->acc2;
    for (; done < npair && A.np < kGrids / 4; ++A.np) {
      XyJob q[4];  // Z, W of T1, then of T3
      std::memset(q, 0, sizeof(q));
      for (int k = 0; k < 2 && done < npair; ++k, ++done) {
        const double* f[4][2] = {{xi(a), xi(b)}, {gx(a), gx(b)}, {xi(a), gx(b)}, {xi(b), gx(a)}};
        for (int j = 0; j < 4; ++j) {
          (k ? q[j].c : q[j].a) = f[j][0];
          (k ? q[j].d : q[j].b) = f[j][1];
        }
        if (++b == nvec) {
          ++a;
          b = a + 1;
        }
      }
      for (int j = 0; j < 4; ++j) {
        q[j].out = m->grid[X.njob];
        X.job[X.njob++] = q[j];
        (j % 2 ? A.w : A.z)[j / 2][A.np] = q[j].out;
      }
    }
    MEAS_CHECK(launch_xy(m, false, X, s));
    MEAS_CHECK((launch_t<false, T_CROSS>(m, 2, A, s)));
  }
  MEAS_CHECK(inv3(m, m->acc, 0, scale, out_dev, s));
  MEAS_CHECK(inv3(m, m->acc2, 0, scale, out_dev + 2 * d, s));
  // T2: (xi_n . Gxi_n) * (xi_m . Gxi_m), n < m: sum_m conj(sum_{n<m} H_n) H_m
  for (int n = 0; n < nvec;) {
    XyArgs X;
    TArgs A;
    std::memset(&X, 0, sizeof(X));
    std::memset(&A, 0, sizeof(A));
    A.first = n == 0;
    A.out[0] = m->acc;
    A.run = m->run;
    for (; n < nvec && A.np < kGrids; ++n, ++A.np) {
      X.job[X.njob++] = XyJob{nullptr, xi(n), gx(n), nullptr, nullptr, m->grid[A.np], nullptr};
      A.z[0][A.np] = m->grid[A.np];
    }
    MEAS_CHECK(launch_xy(m, false, X, s));
    MEAS_CHECK((launch_t<false, T_PREFIX>(m, 1, A, s)));
  }
  MEAS_CHECK(inv3(m, m->acc, 0, scale, out_dev + d, s));
  return FPH_OK;
}

}  // extern "C"
