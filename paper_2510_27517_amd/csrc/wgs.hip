// One-workgroup solver for small stencil systems: a whole PCG solve in one
// launch, with the matrices in registers.
//
// What bounds a small system is one wave's serial instruction stream, not
// memory. Here each thread keeps its rows' values of A, G^T and G and its
// entries of x, r and d in registers for the whole solve; only d, r and t, the
// vectors that neighbouring rows gather, go through LDS, and q, s and the
// gathered r_i - alpha q are formed once by their own row. Every row and every
// inner product is computed as by the iteration kernels (rows in the same order,
// sums that do not depend on their split), so the result is theirs bit for bit. A diagonal's entry that a row
// does not have is a zero times a finite value (LDS is padded with zeros on
// both sides), which adds +0 to a sum that can never be -0.
//
// Threads per workgroup and rows per thread: the reductions cost each wave
// about as much as four of its rows' work, and one workgroup's waves share
// four SIMDs, so few waves with several rows each are best until the values no
// longer fit in registers (launch_wgs). Inside the kernel an iteration takes
// 1.1 us at 64 rows (one wave, no barrier), 1.6 at 256, 2.3 at 1024 and 3.0 at
// 2025 (2D FP64; 3D at 1000 rows 3.2), against 8.9 at 64 and 19 at 1024 rows
// when the matrices are read from memory in every iteration.
//
// Built with floating-point contraction off, like every kernel here.
#include <hip/hip_runtime.h>
#include <cstdint>

#include "device.h"
#include "kernels.h"

namespace pcgk {

namespace {

#define LDSP __attribute__((address_space(3)))

// Totals of NV double-doubles over the NW waves, rounded once, in every
// thread. sh: NV NW slots that no other call uses until two barriers later.
template <int NW>
__device__ __forceinline__ double total1(Acc a, LDSP Acc *sh) {
  a = wave_total(a);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if constexpr (NW == 1) {
    return readlane_f64(a.hi + a.lo, 63);
  } else {
    if (lane == 63) {
      sh[w].hi = a.hi;
      sh[w].lo = a.lo;
    }
    __syncthreads();
    const int q = lane & (NW - 1);
    const Acc v = lanes_total<NW>(Acc{sh[q].hi, sh[q].lo});
    return uniform(v.hi + v.lo);
  }
}
template <int NW>
__device__ __forceinline__ void total2(Acc a, Acc b, double &ta, double &tb, LDSP Acc *sh) {
  const Acc s = wave_total2(a, b);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if constexpr (NW == 1) {
    ta = readlane_f64(s.hi + s.lo, 31);
    tb = readlane_f64(s.hi + s.lo, 63);
  } else {
    if ((lane & 31) == 31) {
      sh[(lane >> 5) * NW + w].hi = s.hi;
      sh[(lane >> 5) * NW + w].lo = s.lo;
    }
    __syncthreads();
    // lanes of the lower half add the first value's waves, the upper the second's
    const int q = (lane >> 5) * NW + (lane & (NW - 1));
    const Acc v = lanes_total<NW>(Acc{sh[q].hi, sh[q].lo});
    ta = readlane_f64(v.hi + v.lo, 0);
    tb = readlane_f64(v.hi + v.lo, 32);
  }
}

// Row r's values at the listed column offsets (ascending) from a matrix in
// sliced diagonals; zero where the row has none. A wave's rows are one slice.
template <typename TV, int W>
__device__ __forceinline__ void load_row(const DevCSR &M, const int32_t (&offs)[W], int count, int r, bool has,
                                         TV (&v)[W]) {
  const int c = __builtin_amdgcn_readfirstlane(r / kSliceRows);
#pragma unroll
  for (int k = 0; k < W; ++k) v[k] = (TV)0;
  if (c >= M.nblk) return;
  GLOBAL const int32_t *blk = gl(M.blk), *off = gl(M.ci);
  const int a = blk[c], e = blk[c + 1];
  for (int p = a; p < e; ++p) {
    const int32_t o = off[p];
    const int64_t at = (int64_t)p * kSliceRows + r % kSliceRows;
    TV x;
    switch (M.dtype) {
      case F64: x = (TV)gl((const double *)M.val)[at]; break;
      case F32: x = (TV)gl((const float *)M.val)[at]; break;
      case BF16: x = (TV)ldval<false>(gl((const bf16_t *)M.val), at); break;
      default: x = (TV)ldval<false>(gl((const _Float16 *)M.val), at); break;
    }
    if (!has) x = (TV)0;
#pragma unroll
    for (int k = 0; k < W; ++k)
      if (k < count && offs[k] == o) v[k] = x;
  }
}

}  // namespace

// WA, WG: diagonals of A and of G and G^T the registers are laid out for
// (unused ones hold zeros at offset 0). NW waves, RPT rows per thread.
template <typename TV, int WA, int WG, int NW, int RPT>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(1, (NW + 3) / 4))) void k_solve_wgs(
    WgsArgs P, State S0) {
  constexpr int NT = NW * 64;
  const uint64_t t0 = __builtin_readsteadycounter();
  __shared__ Acc sh_[6 * NW];
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  LDSP Acc *sh = (LDSP Acc *)sh_;
  const int n = P.n, pad = P.pad, tid = threadIdx.x;
  // [pad zeros | n entries | pad zeros] each
  LDSP TV *dL = (LDSP TV *)dyn_lds + pad, *rL = dL + n + 2 * pad, *tL = rL + n + 2 * pad;
  TV va[RPT][WA], vt[RPT][WG], vg[RPT][WG], x[RPT], r[RPT], d[RPT];
  int32_t oa[WA], ot[WG], og[WG];
#pragma unroll
  for (int k = 0; k < WA; ++k) oa[k] = k < P.na ? P.offA[k] : 0;
#pragma unroll
  for (int k = 0; k < WG; ++k) {
    ot[k] = k < P.nt ? P.offT[k] : 0;
    og[k] = k < P.ng ? P.offG[k] : 0;
  }
  auto has = [&](int j) { return tid + j * NT < n; };
  auto rhs = [&](int j) -> TV {
    const int i = tid + j * NT;
    if (i >= n) return (TV)0;
    return P.io64 ? (TV)gl((const double *)P.b)[i] : gl((const TV *)P.b)[i];
  };
#pragma unroll
  for (int j = 0; j < RPT; ++j) {
    const int i = tid + j * NT;
    load_row<TV, WA>(P.A, oa, P.na, i, has(j), va[j]);
    load_row<TV, WG>(P.GT, ot, P.nt, i, has(j), vt[j]);
    load_row<TV, WG>(P.G, og, P.ng, i, has(j), vg[j]);
    x[j] = (TV)0;
    if (has(j)) x[j] = P.io64 ? (TV)gl((const double *)P.x)[i] : gl((const TV *)P.x)[i];
    r[j] = d[j] = (TV)0;
  }
  for (int i = tid; i < 3 * (n + 2 * pad); i += NT) (dL - pad)[i] = (TV)0;
  __syncthreads();

  auto put = [&](LDSP TV *v, const TV (&a)[RPT]) {
#pragma unroll
    for (int j = 0; j < RPT; ++j)
      if (has(j)) v[tid + j * NT] = a[j];
  };
  auto rows = [&](auto &vals, const auto &offs, LDSP const TV *v, TV (&s)[RPT]) {
    constexpr int W = (int)(sizeof(offs) / sizeof(offs[0]));
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
      const int i = min(tid + j * NT, n - 1);
      TV g[W];
#pragma unroll
      for (int k = 0; k < W; ++k) g[k] = v[i + offs[k]];
      s[j] = (TV)0;
#pragma unroll
      for (int k = 0; k < W; ++k) s[j] += vals[j][k] * g[k];
    }
  };

  const double eps = S0.eps;
  const TV epsv = (TV)eps;
  State o = S0;
  double bb;
  {
    Acc a{0.0, 0.0};
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
      const TV b = rhs(j);
      if (P.keep && has(j)) gl((TV *)P.keep)[tid + j * NT] = b;
      acc_prod(a, b, b);
    }
    bb = total1<NW>(a, sh);
  }
  const double tol_nb = S0.tol * sqrt(bb);
  o.bb = bb;
  o.tol_nb = tol_nb;
  o.alpha = o.beta = 0.0;
  o.restarts = 0;
  auto publish = [&]() {
#pragma unroll
    for (int j = 0; j < RPT; ++j)
      if (has(j)) {
        if (P.io64)
          gl((double *)P.x)[tid + j * NT] = (double)x[j];
        else
          gl((TV *)P.x)[tid + j * NT] = x[j];
      }
    if (tid == 0) {
      o.ticks = (double)(__builtin_readsteadycounter() - t0);
      st_state(gl(P.st), o);
      st_state(gl(P.host), o);
    }
  };
  if (bb == 0.0) {
#pragma unroll
    for (int j = 0; j < RPT; ++j) x[j] = (TV)0;
    o.status = ST_ZERO_B;
    o.done = 1;
    o.iter = 0;
    o.rr = o.tt = o.true_rr = 0.0;
    publish();
    return;
  }
  int it = 0, status = ST_RUNNING;
  double delta = 0.0, rr = 0.0, tt = 0.0, true_rr = 0.0;
  // r = b - A v for the vector v held by rows, gathered through tL
  auto residual = [&](const TV (&v)[RPT]) {
    __syncthreads();
    put(tL, v);
    __syncthreads();
    TV s[RPT];
    rows(va, oa, tL, s);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < RPT; ++j) r[j] = rhs(j) - s[j];
  };
  // t = G^T r into tL, rr and tt (r just formed by rows)
  auto apply_gt = [&]() {
    put(rL, r);
    __syncthreads();
    TV t[RPT];
    rows(vt, ot, rL, t);
    Acc a{0.0, 0.0}, b{0.0, 0.0};
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
      acc_prod(a, r[j], r[j]);
      acc_prod(b, t[j], t[j]);
    }
    put(tL, t);
    if constexpr (NW == 1) __syncthreads();
    total2<NW>(a, b, rr, tt, sh + 2 * NW);
  };
  // s = G t (+ eps r); d = s + beta d
  auto apply_g = [&](TV beta) {
    TV s[RPT];
    rows(vg, og, tL, s);
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
      const TV sv = eps != 0.0 ? s[j] + epsv * r[j] : s[j];
      d[j] = sv + beta * d[j];
    }
    put(dL, d);
    __syncthreads();
  };
  auto restart = [&]() {
    apply_gt();
    const double dn = tt + eps * rr;
    if (sqrt(rr) <= tol_nb)
      status = ST_CONV_REC;
    else if (it >= S0.maxit)
      status = ST_MAXIT;
    delta = dn;
    if (status != ST_RUNNING) return;
    apply_g((TV)0.0);
  };
  residual(x);
  restart();
  for (;;) {
    while (status == ST_RUNNING) {
      TV q[RPT];
      rows(va, oa, dL, q);
      double gamma;
      {
        Acc a{0.0, 0.0};
#pragma unroll
        for (int j = 0; j < RPT; ++j) acc_prod(a, d[j], q[j]);
        gamma = total1<NW>(a, sh);
      }
      if (!(gamma > 0.0) || !isfinite(gamma)) {  // x stays x_i
        status = ST_BREAK_GAMMA;
        break;
      }
      const double alpha = delta / gamma;
      const TV al = (TV)alpha;
      if (S0.rr_period > 0 && it > 0 && it % S0.rr_period == 0) {
        TV v[RPT];  // r_{i+1} = b - A (x_i + alpha_i d_i)
#pragma unroll
        for (int j = 0; j < RPT; ++j) v[j] = x[j] + al * d[j];
        residual(v);
      } else {
#pragma unroll
        for (int j = 0; j < RPT; ++j) r[j] = r[j] - al * q[j];
      }
      apply_gt();
      const double dn = tt + eps * rr;
      const int i1 = it + 1;
      if (!(dn >= 0.0) || !isfinite(dn))
        status = ST_BREAK_DELTA;
      else if (sqrt(rr) <= tol_nb)
        status = ST_CONV_REC;
      else if (i1 >= S0.maxit)
        status = ST_MAXIT;
#pragma unroll
      for (int j = 0; j < RPT; ++j) x[j] = x[j] + al * d[j];
      it = i1;
      if (status != ST_RUNNING) {
        if (status != ST_BREAK_DELTA) delta = dn;
        break;
      }
      const TV beta = (TV)(dn / delta);
      delta = dn;
      apply_g(beta);
    }
    // the true residual b - A x, after a breakdown too
    residual(x);
    {
      Acc a{0.0, 0.0};
#pragma unroll
      for (int j = 0; j < RPT; ++j) acc_prod(a, r[j], r[j]);
      true_rr = total1<NW>(a, sh + 4 * NW);
    }
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
  publish();
}

// Rows the registers hold: eight waves of four rows a thread, but in FP64
// with more than 5 and 3 diagonals (15 values a row) four waves only, beyond
// which the compiler spills.
int32_t wgs_max_n(const Types &ty, int32_t na, int32_t ng) {
  if (ty.vec != ty.a || (ty.vec == F32 && ty.g == F64) || na > kWgsMaxA || ng > kWgsMaxG) return 0;
  return ty.vec == F64 && (na > 5 || ng > 3) ? 1024 : kWgsMaxN;
}

size_t wgs_lds_bytes(int vec_dtype, int32_t n, int32_t pad) {
  return 3 * ((size_t)n + 2 * (size_t)pad) * dtype_size(vec_dtype);
}

template <typename TV, int WA, int WG>
static hipError_t launch_size(const WgsArgs &P, const State &S0, size_t lds, hipStream_t s) {
#define PCG_WGS(NW, RPT) hipLaunchKernelGGL((k_solve_wgs<TV, WA, WG, NW, RPT>), dim3(1), dim3(NW * 64), lds, s, P, S0)
  if (P.n <= 64)
    PCG_WGS(1, 1);
  else if (P.n <= 256)
    PCG_WGS(4, 1);
  else if (P.n <= 512)
    PCG_WGS(4, 2);
  else if (P.n <= 1024)
    PCG_WGS(4, 4);
  else if constexpr (sizeof(TV) == 8 && WA > 5)
    return hipErrorInvalidValue;
  else if (P.n <= 2048)
    PCG_WGS(8, 4);
  else
    return hipErrorInvalidValue;
#undef PCG_WGS
  return hipGetLastError();
}

hipError_t launch_wgs(const Types &ty, const WgsArgs &P, const State &S0, hipStream_t s) {
  if (P.n > wgs_max_n(ty, P.na, P.nt > P.ng ? P.nt : P.ng)) return hipErrorInvalidValue;
  const size_t lds = wgs_lds_bytes(ty.vec, P.n, P.pad);
  const bool narrow = P.na <= 5 && P.nt <= 3 && P.ng <= 3;
  if (ty.vec == F64) return narrow ? launch_size<double, 5, 3>(P, S0, lds, s) : launch_size<double, 7, 4>(P, S0, lds, s);
  return narrow ? launch_size<float, 5, 3>(P, S0, lds, s) : launch_size<float, 7, 4>(P, S0, lds, s);
}

}  // namespace pcgk
