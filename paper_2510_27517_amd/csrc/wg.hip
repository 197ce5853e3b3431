// One-workgroup solver: a whole PCG solve of a small system in one launch
// (the phases, row sums and inner products of the iteration kernels).
// Built with floating-point contraction off, like every kernel here.
#include <hip/hip_runtime.h>
#include <cstdint>

#include "device.h"
#include "kernels.h"

namespace pcgk {

// Totals of a workgroup's double-double sums, rounded once, in every thread.
template <int NV>
__device__ __forceinline__ void wg_totals(Acc (&v)[NV], double (&out)[NV], Acc *sh) {
  reduce_partials<NV>(v, out, sh);
}

// Every row of M by this one workgroup: the eight die-slabs of the
// iteration kernels' partition, one after the other, then a barrier (the
// vector written is read by the next phase). Ordinary loads: a small
// system's matrices stay in L2 from one iteration to the next.
// CSR blocks are staged by the plain loop: in rounds of four entries a thread a
// graph of 9,000 took 220 us per iteration in FP64 and 214 with FP32 vectors
// against 202 and 178, elasticity 12^3 in CSR 934 against 762 with FP32 vectors
// (rounds of eight: 217, 201 and 699, but P P^T of 3,000 64 against 48).
template <typename TACC, int UW, bool REV, typename TM, typename Pre, typename Gather, typename Epi>
__device__ __forceinline__ void wg_rows(const Mat<TM> &M, TACC *lds, Pre pre, Gather gather, Epi epi) {
  for (int l = 0; l < 8; ++l) for_rows_as<TACC, UW, 1, false, REV>(M, l, 8, lds, pre, gather, epi, NoHook{});
  __syncthreads();
}

// Elementwise over all rows by this workgroup, then a barrier.
template <typename F>
__device__ __forceinline__ void wg_elementwise(int n, F f) {
  for (int64_t i = threadIdx.x; i < n; i += kBlock) f(i);
  __syncthreads();
}

// The solve of one system by this workgroup. The iteration vectors x, q, t,
// r (two slots) and d (two slots) are reached through VP: global memory, or
// the workgroup's LDS for a system small enough (then x is copied in and out
// by the kernel). b, the matrices and the state stay in global memory. Both
// placements run the same operations in the same order.
template <typename TV, typename TA, typename TG, bool HAS_EPS, typename VP>
__device__ __forceinline__ void solve_wg(const SysDev &D, GLOBAL State *st, const State &S0, TV *lds, Acc *sh, VP __restrict__ x,
                                         VP __restrict__ q, VP __restrict__ t, VP r0, VP r1, VP d0, VP d1) {
  const int n = D.n;
  const Mat<TA> A = mat<TA>(D.A);
  const Mat<TG> GT = mat<TG>(D.GT), G = mat<TG>(D.G);
  GLOBAL const TV *__restrict__ b = gl((const TV *)D.b);
  VP rv[2] = {r0, r1};
  VP dv[2] = {d0, d1};
  const double eps = S0.eps;
  const TV epsv = (TV)eps;
  // ||b||^2, tol ||b||
  double bb;
  {
    Acc a[1] = {{0.0, 0.0}};
    for (int64_t i = threadIdx.x; i < n; i += kBlock) acc_prod(a[0], b[i], b[i]);
    double v[1];
    wg_totals<1>(a, v, sh);
    bb = v[0];
  }
  const double tol_nb = S0.tol * sqrt(bb);
  State o = S0;
  o.bb = bb;
  o.tol_nb = tol_nb;
  o.alpha = o.beta = 0.0;
  o.restarts = 0;
  if (bb == 0.0) {
    wg_elementwise(n, [&](int64_t i) { x[i] = (TV)0; });
    o.status = ST_ZERO_B;
    o.done = 1;
    o.iter = 0;
    o.rr = o.tt = o.true_rr = 0.0;
    if (threadIdx.x == 0) st_state(st, o);
    return;
  }
  wg_elementwise(n, [&](int64_t i) { dv[0][i] = (TV)0; dv[1][i] = (TV)0; });
  int it = 0;
  int status = ST_RUNNING;
  double delta = 0.0, rr = 0.0, tt = 0.0, true_rr = 0.0;
  // r_it = b - A x (true residual), its norm when `reduce`
  auto residual = [&](VP rout, bool reduce) {
    Acc a[1] = {{0.0, 0.0}};
    wg_rows<TV, 4, false>(
        A, lds, [&](int row) { return RowVals<TV>{b[row], (TV)0, (TV)0}; }, [&](int j) -> TV { return x[j]; },
        [&](int row, TV sum, const RowVals<TV> &pv) {
          const TV r = pv.a - sum;
          rout[row] = r;
          acc_prod(a[0], r, r);
        });
    double v[1];
    wg_totals<1>(a, v, sh);
    if (reduce) true_rr = v[0];
  };
  // start or restart from r_it: t = G^T r, rr, tt, delta, d_it = G t + eps r
  // (beta = 0 against the zeroed or previous direction buffer), stop tests
  auto restart = [&]() {
    const VP src = rv[it & 1];
    Acc a[2] = {{0.0, 0.0}, {0.0, 0.0}};
    wg_rows<TV, 4, true>(
        GT, lds, [&](int row) { return RowVals<TV>{src[row], (TV)0, (TV)0}; }, [&](int j) -> TV { return src[j]; },
        [&](int row, TV sum, const RowVals<TV> &pv) {
          t[row] = sum;
          acc_prod(a[0], pv.a, pv.a);
          acc_prod(a[1], sum, sum);
        });
    double v[2];
    wg_totals<2>(a, v, sh);
    rr = v[0];
    tt = v[1];
    const double dn = tt + eps * rr;
    if (sqrt(rr) <= tol_nb)
      status = ST_CONV_REC;
    else if (it >= S0.maxit)
      status = ST_MAXIT;
    delta = dn;
    if (status != ST_RUNNING) return;
    const VP dnext = dv[it & 1];
    const VP dprev = dv[(it + 1) & 1];
    const TV beta = (TV)0.0;
    wg_rows<TV, 4, false>(
        G, lds, [&](int row) { return RowVals<TV>{HAS_EPS ? src[row] : (TV)0, dprev[row], (TV)0}; },
        [&](int j) -> TV { return t[j]; },
        [&](int row, TV sum, const RowVals<TV> &pv) {
          const TV sv = HAS_EPS ? sum + epsv * pv.a : sum;
          dnext[row] = sv + beta * pv.b;
        });
  };
  residual(rv[0], false);
  restart();
  for (;;) {
    while (status == ST_RUNNING) {
      const VP dcur = dv[it & 1];
      // q = A d_i, gamma = d_i^T q
      double gamma;
      {
        Acc a[1] = {{0.0, 0.0}};
        wg_rows<TV, 8, false>(
            A, lds, [&](int row) { return RowVals<TV>{dcur[row], (TV)0, (TV)0}; },
            [&](int j) -> TV { return dcur[j]; },
            [&](int row, TV sum, const RowVals<TV> &pv) {
              q[row] = sum;
              acc_prod(a[0], pv.a, sum);
            });
        double v[1];
        wg_totals<1>(a, v, sh);
        gamma = v[0];
      }
      if (!(gamma > 0.0) || !isfinite(gamma)) {  // x stays x_i
        status = ST_BREAK_GAMMA;
        break;
      }
      const double alpha = delta / gamma;
      const TV al = (TV)alpha;
      const VP rnext = rv[(it + 1) & 1];
      const bool replace = S0.rr_period > 0 && it > 0 && it % S0.rr_period == 0;
      Acc a[2] = {{0.0, 0.0}, {0.0, 0.0}};
      if (replace) {  // r_{i+1} = b - A (x_i + alpha_i d_i), then t = G^T r_{i+1}
        wg_rows<TV, 4, false>(
            A, lds, [&](int row) { return RowVals<TV>{b[row], (TV)0, (TV)0}; },
            [&](int j) -> TV { return x[j] + al * dcur[j]; },
            [&](int row, TV sum, const RowVals<TV> &pv) { rnext[row] = pv.a - sum; });
        wg_rows<TV, 4, true>(
            GT, lds, [&](int row) { return RowVals<TV>{rnext[row], (TV)0, (TV)0}; },
            [&](int j) -> TV { return rnext[j]; },
            [&](int row, TV sum, const RowVals<TV> &pv) {
              t[row] = sum;
              acc_prod(a[0], pv.a, pv.a);
              acc_prod(a[1], sum, sum);
            });
      } else {  // r_{i+1} = r_i - alpha_i q, formed where it is gathered
        const VP src = rv[it & 1];
        wg_rows<TV, 4, true>(
            GT, lds, [&](int row) { return RowVals<TV>{src[row], q[row], (TV)0}; },
            [&](int j) -> TV { return src[j] - al * q[j]; },
            [&](int row, TV sum, const RowVals<TV> &pv) {
              const TV rn = pv.a - al * pv.b;
              rnext[row] = rn;
              t[row] = sum;
              acc_prod(a[0], rn, rn);
              acc_prod(a[1], sum, sum);
            });
      }
      double v[2];
      wg_totals<2>(a, v, sh);
      rr = v[0];
      tt = v[1];
      const double dn = tt + eps * rr;
      const int i1 = it + 1;
      if (!(dn >= 0.0) || !isfinite(dn))
        status = ST_BREAK_DELTA;
      else if (sqrt(rr) <= tol_nb)
        status = ST_CONV_REC;
      else if (i1 >= S0.maxit)
        status = ST_MAXIT;
      const TV ap = (TV)alpha;
      if (status != ST_RUNNING) {  // x_{i+1} = x_i + alpha_i d_i
        wg_elementwise(n, [&](int64_t i) { x[i] = x[i] + ap * dcur[i]; });
        if (status != ST_BREAK_DELTA) delta = dn;
        it = i1;
        break;
      }
      const TV beta = (TV)(dn / delta);
      delta = dn;
      const VP dnext = dv[i1 & 1];
      wg_rows<TV, 4, false>(
          G, lds, [&](int row) { return RowVals<TV>{HAS_EPS ? rnext[row] : (TV)0, dcur[row], x[row]}; },
          [&](int j) -> TV { return t[j]; },
          [&](int row, TV sum, const RowVals<TV> &pv) {
            const TV sv = HAS_EPS ? sum + epsv * pv.a : sum;
            dnext[row] = sv + beta * pv.b;
            x[row] = pv.c + ap * pv.b;
          });
      it = i1;
    }
    // the true residual b - A x into the current r slot, after a breakdown too
    residual(rv[it & 1], true);
    if (status == ST_CONV_REC && S0.confirm && !(sqrt(true_rr) <= tol_nb)) {
      ++o.restarts;  // the recurrence drifted: restart from the true residual
      status = ST_RUNNING;
      restart();
      continue;
    }
    break;
  }
  o.iter = it;
  o.status = status;
  o.done = 1;
  o.rr = rr;
  o.tt = tt;
  o.delta = delta;
  o.true_rr = true_rr;
  if (threadIdx.x == 0) st_state(st, o);
}

// Iteration vectors in LDS: 7 n values (x, q, t, r0, r1, d0, d1).
#define LDSP __attribute__((address_space(3)))
constexpr int kWgVectors = 7;
// the host sizes the dynamic LDS assuming at most this much static LDS
static_assert(kLdsBytes + 4 * (kBlock / 64) * sizeof(Acc) + 2 * 8 * sizeof(double) <= kWgStaticLdsBytes,
              "static LDS of the one-workgroup solver");

// One workgroup per system of the set solves it whole. lds_vec_bytes: the
// dynamic LDS of the launch; a system whose seven iteration vectors fit in it
// keeps them there (a phase's gathers and stores then stay on the CU instead
// of going through L2), any other keeps them in global memory.
template <typename TV, typename TA, typename TG, bool HAS_EPS>
__global__ __launch_bounds__(kBlock) void k_solve_wg(const SysDev *__restrict__ dir, const int32_t *__restrict__ set,
                                                     int lds_vec_bytes) {
  __shared__ TV lds[kLdsBytes / sizeof(TV)];
  __shared__ Acc sh[4 * (kBlock / 64)];
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  const SysDev &D = dir[set[blockIdx.x]];
  GLOBAL State *st = gl(D.st);
  const State S0 = ld_state(st);
  const int n = D.n;
  GLOBAL TV *__restrict__ xg = gl((TV *)D.x);
  if ((int64_t)kWgVectors * n * (int64_t)sizeof(TV) <= lds_vec_bytes) {
    LDSP TV *v = (LDSP TV *)dyn_lds;
    wg_elementwise(n, [&](int64_t i) { v[i] = xg[i]; });
    solve_wg<TV, TA, TG, HAS_EPS>(D, st, S0, lds, sh, v, v + n, v + 2 * n, v + 3 * n, v + 4 * n, v + 5 * n,
                                  v + 6 * n);
    __syncthreads();
    for (int64_t i = threadIdx.x; i < n; i += kBlock) xg[i] = v[i];
  } else {
    solve_wg<TV, TA, TG, HAS_EPS>(D, st, S0, lds, sh, xg, gl((TV *)D.q), gl((TV *)D.t), gl((TV *)D.r0),
                                  gl((TV *)D.r1), gl((TV *)D.d0), gl((TV *)D.d1));
  }
}

bool solve_wg_supported(const Types &ty) {
  return (ty.vec == F64 && ty.a == F64 && ty.g == F64) ||
         (ty.vec == F32 && ty.a == F32 && (ty.g == F32 || ty.g == BF16 || ty.g == F16));
}

hipError_t launch_solve_wg(const Types &ty, const LaunchSet &L, bool has_eps, hipStream_t s) {
  if (L.nset == 0) return hipSuccess;
#define PCG_SOLVE_WG(TV, TG)                                                                                   \
  do {                                                                                                         \
    if (has_eps)                                                                                               \
      hipLaunchKernelGGL((k_solve_wg<TV, TV, TG, true>), dim3(L.nset), dim3(kBlock), vec_bytes, s, L.dir,      \
                         L.set, vec_bytes);                                                                    \
    else                                                                                                       \
      hipLaunchKernelGGL((k_solve_wg<TV, TV, TG, false>), dim3(L.nset), dim3(kBlock), vec_bytes, s, L.dir,     \
                         L.set, vec_bytes);                                                                    \
  } while (0)
  if (!solve_wg_supported(ty)) return hipErrorInvalidValue;
  const int vec_bytes = ty.vec == F64 ? kWgVectors * 8 * L.wg_lds_rows8 : kWgVectors * 4 * L.wg_lds_rows4;
  if (ty.vec == F64)
    PCG_SOLVE_WG(double, double);
  else if (ty.g == F32)
    PCG_SOLVE_WG(float, float);
  else if (ty.g == BF16)
    PCG_SOLVE_WG(float, bf16_t);
  else
    PCG_SOLVE_WG(float, _Float16);
#undef PCG_SOLVE_WG
  return hipGetLastError();
}

}  // namespace pcgk
