// The whole (P)CG solve of a small system in one launch: one workgroup per
// right-hand side runs the slots of fph_solve.h one after the other.
//
// A slot of a small system is two or four launches of a few workgroups whose
// time is launches, memory round trips and the state's folds; inside one
// workgroup the same phases (the operator sweep, the update, the transforms
// and series of fph_batch_pc.h) follow each other through barriers, and the
// vectors stay in the compute unit's caches.  Every decision is taken by the
// functions of fph_common.h on a state of the same form, so a solve takes the
// same path as the launch sequence up to the order of its sums.  Bound by its
// chain of phases: L = 4, Ltau = 40, preconditioned FP64 takes 15 us per
// iteration against 26 us in four launches (without: 4.4 against 11 us).
#pragma once

#include "fph_batch.h"
#include "fph_solve.h"

namespace fph {

constexpr int kSmallNT = 512;
constexpr size_t kSmallLds = (size_t)156 << 10;  // LDS a workgroup may take

template <typename TI>
struct SmallArgs {
  SlotArgs<TI> s;
  TI* uit;                       // what the update advances: u_dev, or the FP32 correction
  PcView<TI> pc;                 // of field 0
  int pre, zero;
  long total;                    // slots: 1 + maxiter + max_outer
  SolveInit init;
};

// LDS bytes: the transforms' tables, r and, preconditioned, z and the transform
// workspace (a memory round trip costs some 1 000 cycles here), kept for the
// whole solve; then the larger of four FP64 slices per chunk of the sweep, the transforms' tiles and the
// series' buffers.
template <typename TI>
size_t small_lds(const Geom& g, int H1, int H2, bool pre) {
  const int S = (g.Q <= kSmallNT) ? kSmallNT / g.Q : 1, H = H1 * H2;
  size_t lds = 4 * (size_t)S * g.N * sizeof(double);
  if (!pre) return lds + g.d * sizeof(TI);
  constexpr int elem = 2 * sizeof(TI);
  const long tf = bpc_lds_tf(H, bpc_tile_log2(g.N, H, kBpcLdsAlone, elem));
  const long se = bpc_groups(g.L, H, kSmallNT, kBpcLdsAlone, elem) * bpc_lds_series(g.L);
  const size_t pc = (size_t)(tf > se ? tf : se) * elem;
  return (lds > pc ? lds : pc) + (size_t)bpc_lds_tables(H1, H2) * elem + 3 * g.d * sizeof(TI);
}

// Launch: grid nrhs, kSmallNT threads, small_lds bytes.
template <typename TI>
__global__ void __launch_bounds__(kSmallNT)
k_small_solve(Geom g, SmallArgs<TI> a, PcgStatsDev* __restrict__ stats) {
  constexpr int NT = kSmallNT;
  using T2 = typename Cplx<TI>::type;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ double red_sh[NT / 64];
  __shared__ RhsState s_sh;
  T2* tab = reinterpret_cast<T2*>(smem_raw);
  T2* Z = tab + (a.pre ? bpc_lds_tables(a.pc.H1, a.pc.H2) : 0);  // [H][N]: d values
  TI* r = reinterpret_cast<TI*>(Z) + (a.pre ? g.d : 0);
  TI* z = a.pre ? r + g.d : r;
  unsigned char* lds = reinterpret_cast<unsigned char*>(z + g.d);
  const int rh = blockIdx.x;
  const int f = field_of(g, rh);
  const long base = (long)rh * g.d, fo = field_off(g, rh);
  const int tid = threadIdx.x;
  a.pc.info += f;
  a.pc.np += (long)f * g.Ltau;
  a.pc.coef += (long)f * a.pc.H * kNPMax;
  a.pc.dbar += (long)f * g.N;
  a.s.pa += base;
  a.s.pb += base;
  a.s.Ap += base;
  a.s.b += base;
  a.s.u += base;
  a.s.u64b += base;
  a.s.u32 += base;
  a.uit += base;
  int S, sub, lane, nslot;
  block_layout<NT>(g, tid, S, sub, lane, nslot);
  const int Tch = (g.Ltau + S - 1) / S;
  const int tau0 = sub * Tch;
  const bool active = (sub < S) && (tau0 < g.Ltau);
  const int Tc = active ? min(Tch, g.Ltau - tau0) : 0;
  const long lo = 4L * (sub < S ? sub : 0) * g.N;
  auto no_hook = [] { return true; };
  // Adds a reduction to the state as apply_pending does; sums over the block.
  auto fold = [&](int kind, double v, double v2) {
    v = block_sum<NT>(v, red_sh);
    if (kind == P_RES) v2 = block_sum<NT>(v2, red_sh);
    if (tid == 0) apply_pending(s_sh, kind, v, v2, a.pre);
    __syncthreads();
  };

  if (a.pre) bpc_tables<TI, NT>(a.pc, tab);
  if (tid == 0) solve_init_state(s_sh, a.init);
  if (a.zero)
    for (long k = 4L * tid; k < g.d; k += 4L * NT)
      Vec4<double>::st(a.s.u + k, Vec4<double>::V{0.0, 0.0, 0.0, 0.0});
  __syncthreads();
  for (long slot = 0; slot < a.total && !s_sh.final_; ++slot) {
    double acc = 0.0, acc2 = 0.0;
    if (s_sh.replace) {
      EpiResidual<TI> epi{a.s.b, r};
      double* lds4 = reinterpret_cast<double*>(lds) + lo;
      if constexpr (sizeof(TI) == 4) {
        InResid in{a.s.u, a.s.u64b, a.s.u32, nullptr, nullptr, 0};
        in.begin(s_sh);
        mtm_sweep<double, NT, 1, 1>(opaque(g), a.s.E64 + fo, a.s.th64, Tch, tau0, Tc, active, lane, nslot, lds4,
                                    0, in, epi, acc, acc2, no_hook);
      } else {
        InPlain<double> in{a.s.u};
        mtm_sweep<double, NT, 1, 1>(opaque(g), a.s.E64 + fo, a.s.th64, Tch, tau0, Tc, active, lane, nslot, lds4,
                                    0, in, epi, acc, acc2, no_hook);
      }
      fold(P_RES, acc, acc2);
    } else {
      InPUpdate<TI, false> in{z, a.s.pa, a.s.pb, nullptr, nullptr, (TI)0, 0};
      EpiDot<TI> epi{a.s.Ap};
      in.begin(s_sh);
      mtm_sweep<TI, NT, 1, 1>(opaque(g), a.s.E + fo, a.s.th, Tch, tau0, Tc, active, lane, nslot,
                              reinterpret_cast<TI*>(lds) + lo, 0, in, epi, acc, acc2, no_hook);
      acc = block_sum<NT>(acc, red_sh);
      if (tid == 0) {
        InPUpdate<TI, false>::on_state(s_sh);
        apply_pending(s_sh, P_PAP, acc, 0.0, a.pre);
      }
      __syncthreads();
      if (s_sh.done) continue;  // breakdown
      const TI alpha = (TI)s_sh.alpha;
      const bool uz = s_sh.u32z != 0;
      const TI* p = (s_sh.iter & 1) ? a.s.pa : a.s.pb;
      const TI* Ap = a.s.Ap;
      TI* u = a.uit;
      double rr = 0.0;
      for (long k = 4L * tid; k < g.d; k += 4L * NT) {
        auto uu = Vec4<TI>::ld(u + k), rv = Vec4<TI>::ld(r + k);
        const auto pp = Vec4<TI>::ld(p + k), aa = Vec4<TI>::ld(Ap + k);
        if (uz) uu = typename Vec4<TI>::V{};
        uu.x += alpha * pp.x; uu.y += alpha * pp.y; uu.z += alpha * pp.z; uu.w += alpha * pp.w;
        rv.x -= alpha * aa.x; rv.y -= alpha * aa.y; rv.z -= alpha * aa.z; rv.w -= alpha * aa.w;
        Vec4<TI>::st(u + k, uu);
        Vec4<TI>::st(r + k, rv);
        rr += (double)rv.x * (double)rv.x + (double)rv.y * (double)rv.y + (double)rv.z * (double)rv.z +
              (double)rv.w * (double)rv.w;
      }
      rr = block_sum<NT>(rr, red_sh);
      if (tid == 0) {
        s_sh.u32z = 0;
        apply_pending(s_sh, P_RR, rr, 0.0, a.pre);
      }
      __syncthreads();
    }
    if (!a.pre || s_sh.done) continue;
    T2* l = reinterpret_cast<T2*>(lds);
    bpc_forward<TI, NT, kBpcLdsAlone>(opaque(g), a.pc, r, Z, tab, l);
    bpc_series<TI, NT, kBpcLdsAlone>(opaque(g), a.pc, a.s.th, Z, l);
    fold(P_RZ,
         bpc_inverse<TI, NT, kBpcLdsAlone>(opaque(g), a.pc, Z, r, z, tab, l), 0.0);
  }

  // The solution and S_F = b . u (as k_solve_final), then the statistics.
  const bool zero = s_sh.started && s_sh.bb == 0.0;
  const bool from_ws = s_sh.refined && s_sh.upar == 1, add32 = s_sh.refined && !s_sh.u32z;
  double act = 0.0;
  for (long k = 4L * tid; k < g.d; k += 4L * NT) {
    auto uu = Vec4<double>::ld((from_ws ? a.s.u64b : a.s.u) + k);
    if (add32) {
      const float4 c = Vec4<float>::ld(a.s.u32 + k);
      uu.x += (double)c.x; uu.y += (double)c.y; uu.z += (double)c.z; uu.w += (double)c.w;
    }
    if (zero) uu = Vec4<double>::V{0.0, 0.0, 0.0, 0.0};
    if (zero || from_ws || add32) Vec4<double>::st(a.s.u + k, uu);
    const auto bv = Vec4<double>::ld(a.s.b + k);
    act += bv.x * uu.x + bv.y * uu.y + bv.z * uu.z + bv.w * uu.w;
  }
  act = block_sum<NT>(act, red_sh);
  if (tid == 0) stats[rh] = solve_stats(s_sh, act);
}

}  // namespace fph
