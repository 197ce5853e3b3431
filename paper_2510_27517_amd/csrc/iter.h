// The three kernels of a CG iteration over the general layouts, as templates.
// FMT = -1 (kernels.hip): any layout, for launches over many systems; FMT >= 0
// (single.hip): one layout, for a single system. A kernel for all layouts gives
// each the registers and the schedule of the others, which never meet in a
// single system's launch, so a change for one layout moved the others; built
// apart, each takes what is best for it (per iteration, FP64, with the loads of
// single.hip: 3x3 blocks of elasticity 40^3 60.5 -> 59.8 us, a graph of 150,001
// 27.1 -> 26.6 and of 600,001 55.0 -> 51.7, irregular rows of 18,000 23.5 -> 22.4;
// FP32 with a BF16 G: 36.2 -> 36.3, 21.9 -> 21.3, 46.9 -> 43.9, 24.1 -> 23.5).
#pragma once
#include <hip/hip_runtime.h>
#include <cmath>
#include <cstdint>

#include "device.h"
#include "kernels.h"

namespace pcgk {

// UW: loads in flight per lane in the one-row sliced walks (rows longer
// than 4 entries), a tuning knob.
template <typename TV, typename TA, int UW, int FMT = -1>
__global__ __launch_bounds__(kBlock) PCG_OCCUPANCY void k_iter_A(const SysDev *__restrict__ dir,
                                                                 const int2 *__restrict__ map, SysDev one) {
  // staged products in flight per thread: eight in FP64 (A-kernel of a graph of
  // 600,001: 19.4 -> 15.9 us, of 150,001: 7.7 -> 6.9), but in FP32 the plain
  // loop is faster (15.6 against 16.3 us, 5.5 against 5.9)
  constexpr int US = FMT < 0 ? 0 : sizeof(TV) == 8 ? 8 : 1;
  __shared__ TV lds[kLdsBytes / sizeof(TV)];
  __shared__ Acc sh[4 * (kBlock / 64)];
  const Work wk = work_of(dir, map, one);
  const SysDev &D = wk.D;
  const int l = wk.l;
  GLOBAL const State &S = gl(D.st)[0];
  if (S.done) return;
  const Mat<TA> A = mat<TA, FMT>(D.A);
  const int it = S.iter;
  GLOBAL TV *__restrict__ q = gl((TV *)D.q);
  GLOBAL const TV *__restrict__ dcur = gl((const TV *)((it & 1) ? D.d1 : D.d0));  // d_i
  Acc part[1] = {{0.0, 0.0}};
  // pre's d_i[row] is the operand of A's diagonal
  for_rows<TV, UW, US, false, true>(
      A, l, D.A.grid, lds, [&](int row) { return RowVals<TV>{dcur[row], (TV)0, (TV)0}; },
      [&](int j) -> TV { return dcur[j]; },
      [&](int row, TV sum, const RowVals<TV> &pv) {
        q[row] = sum;
        acc_prod(part[0], pv.a, sum);
      });
  put_partials<1>(part, gl(D.pg), part_slot(l, D.A.grid), D.A.grid, sh);
}

template <typename TV, typename TG, int FMT = -1>
__global__ __launch_bounds__(kBlock) PCG_GT_OCCUPANCY void k_iter_GT(const SysDev *__restrict__ dir, const int2 *__restrict__ map, SysDev one,
                                                    int mode) {
  constexpr int US = FMT >= 0 ? 8 : 0;  // staged products in flight: 8.3 -> 8.0 us on 18,000 irregular rows
  __shared__ TV lds[kLdsBytes / sizeof(TV)];
  __shared__ Acc sh[4 * (kBlock / 64)];
  const Work wk = work_of(dir, map, one);
  const SysDev &D = wk.D;
  const int l = wk.l;
  GLOBAL State *st = gl(D.st);
  GLOBAL const State &S = st[0];
  Acc g[1];
  load_partials<1>(gl(D.pg), D.A.grid, g);  // in flight while the state is read
  if (S.done) {  // stopped earlier: st[1] mirrors st[0], so the G-kernel need not read st[0]
    if (l == 0 && threadIdx.x == 0) st_state(st + 1, ld_state(&S));
    return;
  }
  const int it = S.iter;
  if (mode == 3) mode = (S.rr_period > 0 && it > 0 && it % S.rr_period == 0) ? 1 : 0;
  const double delta = S.delta, alpha0 = S.alpha, gamma0 = S.gamma;
  const Mat<TG> GT = mat<TG, FMT>(D.GT);
  GLOBAL const TV *__restrict__ q = gl((const TV *)D.q);
  GLOBAL TV *__restrict__ t = gl((TV *)D.t);
  GLOBAL const TV *__restrict__ src = gl((const TV *)((((mode == 1) ? it + 1 : it) & 1) ? D.r1 : D.r0));
  GLOBAL TV *__restrict__ dst = gl((TV *)(((it + 1) & 1) ? D.r1 : D.r0));
  // alpha_i = delta_i / gamma_i (published in st[1] after the walk); false
  // on breakdown
  double alpha = alpha0, gamma = gamma0;
  bool brk = false;
  TV al = (TV)0;
  auto step = [&]() -> bool {
    if (mode != 2) {
      double gv[1];
      reduce_partials<1>(g, gv, sh);
      gamma = gv[0];
      brk = !(gamma > 0.0) || !isfinite(gamma);
      alpha = brk ? 0.0 : delta / gamma;  // on breakdown x already holds x_i
    }
    al = (mode == 0) ? (TV)alpha : (TV)0;
    return !brk;
  };
  auto publish = [&]() {
    if (l == 0 && threadIdx.x == 0) {
      State o = ld_state(&S);
      o.gamma = gamma;
      o.alpha = alpha;
      if (brk) {
        o.status = ST_BREAK_GAMMA;
        o.done = 1;
      }
      st_state(st + 1, o);
    }
  };
  Acc part[2] = {{0.0, 0.0}, {0.0, 0.0}};
  // each die walks its slices from the top down (measured slightly faster);
  // two rows per lane over sliced diagonals where the operand is the
  // difference of two gathered vectors (the other kernels, with one, are
  // faster one row per lane), with the first slice pair's loads in flight
  // while alpha is reduced
  if (mode == 0 && rows2(GT)) {
    const int32_t n = GT.n;
    struct PV {
      Pair<TV> s, q;
    };
    // pre2's pair equals gather_pair at offset 0 on every row that exists
    const bool go = for_rows2<TV, true, true>(
        GT, l, D.GT.grid,
        [&](int r0, bool h0, bool h1) -> PV {
          PV o{{(TV)0, (TV)0}, {(TV)0, (TV)0}};
          if (h1) {
            o.s = ld_pair(src, r0);
            o.q = ld_pair(q, r0);
          } else if (h0) {
            o.s.x = src[r0];
            o.q.x = q[r0];
          }
          return o;
        },
        [&](int32_t j0) -> PV { return PV{gather_pair(src, j0, n), gather_pair(q, j0, n)}; },
        [&](const PV &v) -> Pair<TV> { return Pair<TV>{v.s.x - al * v.q.x, v.s.y - al * v.q.y}; },
        [&](int r0, bool h0, bool h1, TV s0, TV s1, const PV &pv) {
          const TV ra = pv.s.x - al * pv.q.x, rb = pv.s.y - al * pv.q.y;
          if (h1) {
            st_pair(dst, r0, ra, rb);
            st_pair(t, r0, s0, s1);
            acc_prod(part[0], ra, ra);
            acc_prod(part[1], s0, s0);
            acc_prod(part[0], rb, rb);
            acc_prod(part[1], s1, s1);
          } else if (h0) {
            dst[r0] = ra;
            t[r0] = s0;
            acc_prod(part[0], ra, ra);
            acc_prod(part[1], s0, s0);
          }
        },
        step);
    publish();
    if (!go) return;
  } else if (!step()) {
    publish();
    return;
  } else if (mode == 0) {
    publish();
    for_rows<TV, 4, US, true>(
        GT, l, D.GT.grid, lds, [&](int row) { return RowVals<TV>{src[row], q[row], (TV)0}; },
        [&](int j) -> TV { return src[j] - al * q[j]; },
        [&](int row, TV sum, const RowVals<TV> &pv) {
          const TV rn = pv.a - al * pv.b;
          dst[row] = rn;
          t[row] = sum;
          acc_prod(part[0], rn, rn);
          acc_prod(part[1], sum, sum);
        });
  } else {
    publish();
    for_rows<TV, 4, US, true>(
        GT, l, D.GT.grid, lds, [&](int row) { return RowVals<TV>{src[row], (TV)0, (TV)0}; },
        [&](int j) -> TV { return src[j]; },
        [&](int row, TV sum, const RowVals<TV> &pv) {
          t[row] = sum;
          acc_prod(part[0], pv.a, pv.a);
          acc_prod(part[1], sum, sum);
        });
  }
  put_partials<2>(part, gl(D.prt), part_slot(l, D.GT.grid), D.GT.grid, sh);
}

template <typename TV, typename TG, bool HAS_EPS, int FMT = -1>
__global__ __launch_bounds__(kBlock) PCG_G_OCCUPANCY void k_iter_G(const SysDev *__restrict__ dir, const int2 *__restrict__ map, SysDev one,
                                                   int mode,
                                                   uint64_t *report) {
  // more in flight per lane, and the first products formed under the reduction of
  // the partial sums (a graph of 150,001, FP32: 6.8 -> 6.4 us; 18,000 irregular
  // rows 6.5 -> 6.1); over 3x3 blocks the reduction stays before the walk
  constexpr int US = FMT >= 0 ? 8 : 0;
  constexpr int UW = FMT >= 0 ? 8 : 4;
  __shared__ TV lds[kLdsBytes / sizeof(TV)];
  __shared__ Acc sh[4 * (kBlock / 64)];
  const Work wk = work_of(dir, map, one);
  const SysDev &D = wk.D;
  const int l = wk.l;
  GLOBAL State *st = gl(D.st);
  // st[1] is the G^T-kernel's publication for this iteration; st[0] is written
  // below by workgroup 0 and must not be read by the others
  GLOBAL const State &S = st[1];
  Acc va[2];
  load_partials<2>(gl(D.prt), D.GT.grid, va);  // in flight while the state is read
  if (S.done) {  // stopped earlier, or the G^T-kernel flagged a breakdown
    if (l == 0 && threadIdx.x == 0) {
      const State o = ld_state(&S);
      st_state(st, o);
      report_progress(report, o.iter, o.done);
    }
    return;
  }
  const int it = S.iter;
  const double delta = S.delta, eps_d = S.eps, tol_nb = S.tol_nb;
  const int maxit = S.maxit;
  const int i1 = (mode == 2) ? it : it + 1;
  // x_{i+1} = x_i + alpha_i d_i (not at a start or restart, mode 2)
  const bool upd = mode != 2;
  const TV ap = (TV)S.alpha;
  GLOBAL TV *__restrict__ x = gl((TV *)D.x);
  GLOBAL const TV *dprev = gl((const TV *)((i1 & 1) ? D.d0 : D.d1));  // d_i (may be d_{i+1}'s buffer)
  // s = G t + eps r, and the next direction d_{i+1} = s + beta d_i (at a
  // start or restart beta = 0, d = s)
  const Mat<TG> G = mat<TG, FMT>(D.G);
  GLOBAL const TV *__restrict__ t = gl((const TV *)D.t);
  GLOBAL const TV *__restrict__ rc = gl((const TV *)((i1 & 1) ? D.r1 : D.r0));
  GLOBAL TV *dnext = gl((TV *)((i1 & 1) ? D.d1 : D.d0));
  const TV eps = (TV)eps_d;
  // delta_{i+1}, beta_i and the stopping tests, published in st[0]; false
  // once the solve stops (then only x is updated)
  TV beta = (TV)0;
  double rr = 0.0, tt = 0.0, dn = 0.0;
  int status = ST_RUNNING;
  auto step = [&]() -> bool {
    double v[2];
    reduce_partials<2>(va, v, sh);
    rr = v[0];
    tt = v[1];
    dn = tt + eps_d * rr;
    if (mode != 2 && (!(dn >= 0.0) || !isfinite(dn)))
      status = ST_BREAK_DELTA;
    else if (sqrt(rr) <= tol_nb)
      status = ST_CONV_REC;
    else if (i1 >= maxit)
      status = ST_MAXIT;
    beta = (TV)((mode == 2) ? 0.0 : dn / delta);
    return status == ST_RUNNING;
  };
  // the first slice's products are formed while the partials are reduced;
  // two rows per lane over sliced diagonals (as in the G^T-kernel: one
  // access of twice the width for each operand, value and result), one
  // otherwise and at a start or restart
  bool go;
  if (upd && rows2(G)) {
    const int32_t n = G.n;
    struct PV {
      Pair<TV> r, d, x;
    };
    go = for_rows2<TV, false, false>(
        G, l, D.G.grid,
        [&](int r0, bool h0, bool h1) -> PV {
          PV o{{(TV)0, (TV)0}, {(TV)0, (TV)0}, {(TV)0, (TV)0}};
          if (h1) {
            if (HAS_EPS) o.r = ld_pair(rc, r0);
            o.d = ld_pair(dprev, r0);
            o.x = ld_pair(x, r0);
          } else if (h0) {
            if (HAS_EPS) o.r.x = rc[r0];
            o.d.x = dprev[r0];
            o.x.x = x[r0];
          }
          return o;
        },
        [&](int32_t j0) -> Pair<TV> { return gather_pair(t, j0, n); },
        [&](const Pair<TV> &v) -> Pair<TV> { return v; },
        [&](int r0, bool h0, bool h1, TV s0, TV s1, const PV &pv) {
          const TV sv0 = HAS_EPS ? s0 + eps * pv.r.x : s0, sv1 = HAS_EPS ? s1 + eps * pv.r.y : s1;
          const TV dn0 = sv0 + beta * pv.d.x, dn1 = sv1 + beta * pv.d.y;
          const TV x0 = pv.x.x + ap * pv.d.x, x1 = pv.x.y + ap * pv.d.y;
          if (h1) {
            st_pair(dnext, r0, dn0, dn1);
            st_pair(x, r0, x0, x1);
          } else if (h0) {
            dnext[r0] = dn0;
            x[r0] = x0;
          }
        },
        step);
  } else if (upd)
    go = for_rows_h<TV, UW, US, (FMT >= 0)>(
        G, l, D.G.grid, lds,
        [&](int row) { return RowVals<TV>{HAS_EPS ? rc[row] : (TV)0, dprev[row], x[row]}; },
        [&](int j) -> TV { return t[j]; },
        [&](int row, TV sum, const RowVals<TV> &pv) {
          const TV sv = HAS_EPS ? sum + eps * pv.a : sum;
          dnext[row] = sv + beta * pv.b;
          x[row] = pv.c + ap * pv.b;
        },
        step);
  else
    go = for_rows_h<TV, UW, US, (FMT >= 0)>(
        G, l, D.G.grid, lds, [&](int row) { return RowVals<TV>{HAS_EPS ? rc[row] : (TV)0, dprev[row], (TV)0}; },
        [&](int j) -> TV { return t[j]; },
        [&](int row, TV sum, const RowVals<TV> &pv) {
          const TV sv = HAS_EPS ? sum + eps * pv.a : sum;
          dnext[row] = sv + beta * pv.b;
        },
        step);
  if (l == 0 && threadIdx.x == 0) {
    State o = ld_state(&S);
    o.rr = rr;
    o.tt = tt;
    o.iter = i1;
    o.alpha = 0.0;  // x += alpha_i d_i is applied in this kernel, whatever the status
    if (status != ST_BREAK_DELTA) {
      o.beta = (mode == 2) ? 0.0 : dn / delta;
      o.delta = dn;
    }
    if (status != ST_RUNNING) {
      o.status = status;
      o.done = 1;
    }
    st_state(st, o);
    report_progress(report, o.iter, o.done);
  }
  if (!go && upd) {  // stopped: x_{i+1} only
    int64_t i0, i1r;
    ew_rows(D.n, l, D.G.grid, i0, i1r);
    for (int64_t i = i0 + threadIdx.x; i < i1r; i += kBlock) x[i] = x[i] + ap * dprev[i];
  }
}

}  // namespace pcgk
