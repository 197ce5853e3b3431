// gfx950 kernels for preconditioned CG with M^-1 = G G^T + eps I.
//
// Every operator product is a sparse matrix-vector product in one of three
// layouts (DevCSR): sliced ELL (a wave owns slices of 64 rows, one lane per
// row, coalesced column and value loads, 32- or 16-bit column indices),
// sliced 3x3 blocks (one index per block), or CSR row blocks (a workgroup
// stages the products of a block of rows in LDS, then one thread per row
// adds them). In every layout each row's products are added left to right
// from zero in CSR order. Matrix loads are nontemporal, or ordinary for a
// matrix kept resident in the memory-side cache (DevCSR::temporal). The A,
// G^T and G products carry the CG vector updates in their gathers and
// epilogues, so one iteration is three launches:
//   A-kernel : q = A d_i,  partials of gamma = d_i^T q;
//   G^T-kernel: alpha_i = delta_i / gamma,
//              r_{i+1} = r_i - alpha_i q  (formed where it is gathered),
//              t = G^T r_{i+1}, partials of ||r||^2, ||t||^2;
//   G-kernel : delta_{i+1} = ||t||^2 + eps ||r||^2 (= r^T M^-1 r),
//              beta_{i+1} = delta_{i+1} / delta_i, convergence test,
//              x_{i+1} = x_i + alpha_i d_i (also on the last iteration),
//              d_{i+1} = (G t + eps r_{i+1}) + beta_{i+1} d_i.
// That is 11 vector streams of n entries per iteration: A reads d, writes
// q; G^T reads r and q, writes r and t; G reads t, d and x, writes x and d.
// d and r alternate between two buffers by iteration parity, so no
// workgroup overwrites a vector entry another one still gathers.
//
// Reductions are deterministic and need no atomics: each workgroup reduces
// its rows with wave shuffles and LDS and writes one partial per value; every
// workgroup of the next kernel adds all partials in the same fixed order
// (kernel boundaries make them visible), so all obtain the identical total.
// One workgroup publishes the updated scalars into a state slot that the
// kernel itself does not read.
//
// Work placement: each of the 8 XCDs (workgroup b runs on XCD b % 8) owns a
// contiguous eighth of the slices (or row blocks), and its workgroups take
// them interleaved, so at any moment an XCD works on one window of
// consecutive rows whose gathered neighbourhoods stay in that XCD's L2.
//
// Built with floating-point contraction off: every product and sum rounds
// separately, in the order written (rows summed left to right from zero),
// which is also the order of the plain CSR definition.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <cmath>
#include <cstdint>
#include <mutex>
#include <type_traits>

#include "device.h"
#include "iter.h"
#include "kernels.h"

namespace pcgk {

// ------------------------------------------------------------------ kernels

template <typename TV, typename TA>
__global__ __launch_bounds__(kBlock) PCG_OCCUPANCY void k_resid(const SysDev *__restrict__ dir, const int2 *__restrict__ map, SysDev one,
                                                  int slot_sel, int with_d, int reduce, int respect_done) {
  __shared__ TV lds[kLdsBytes / sizeof(TV)];
  __shared__ Acc sh[4 * (kBlock / 64)];
  const Work wk = work_of(dir, map, one);
  const SysDev &D = wk.D;
  const int l = wk.l;
  GLOBAL const State &S = gl(D.st)[0];
  if (respect_done && S.done) return;
  const int it = S.iter;
  if (slot_sel == 2) {  // replacement decided per system
    if (!(S.rr_period > 0 && it > 0 && it % S.rr_period == 0)) return;
    slot_sel = 1;
  }
  const Mat<TA> A = mat<TA>(D.A);
  GLOBAL const TV *__restrict__ b = gl((const TV *)D.b);
  GLOBAL const TV *__restrict__ x = gl((const TV *)D.x);
  GLOBAL TV *__restrict__ rout = gl((TV *)(((it + slot_sel) & 1) ? D.r1 : D.r0));
  GLOBAL const TV *__restrict__ dc = gl((const TV *)((it & 1) ? D.d1 : D.d0));  // d_i
  TV al = (TV)0;
  if (with_d) {
    double g[1];
    sum_partials<1>(gl(D.pg), D.A.grid, g, sh);
    if (!(g[0] > 0.0) || !isfinite(g[0])) return;  // the G^T-kernel reports the breakdown
    al = (TV)(S.delta / g[0]);
  }
  Acc part[1] = {{0.0, 0.0}};
  auto pre = [&](int row) { return RowVals<TV>{b[row], (TV)0, (TV)0}; };
  auto epi = [&](int row, TV sum, const RowVals<TV> &pv) {
    const TV rv = pv.a - sum;
    rout[row] = rv;
    acc_prod(part[0], rv, rv);
  };
  if (with_d)
    for_rows<TV>(A, l, D.A.grid, lds, pre, [&](int j) -> TV { return x[j] + al * dc[j]; }, epi);
  else
    for_rows<TV>(A, l, D.A.grid, lds, pre, [&](int j) -> TV { return x[j]; }, epi);
  if (reduce) put_partials<1>(part, gl(D.ptr), part_slot(l, D.A.grid), D.A.grid, sh);
}

template <typename TV>
__global__ __launch_bounds__(kBlock) void k_zero_dirs(const SysDev *__restrict__ dir, const int2 *__restrict__ map,
                                                      int zero_x) {
  const int2 m = map[blockIdx.x];
  const SysDev &D = dir[m.x];
  GLOBAL TV *__restrict__ d0 = gl((TV *)D.d0);
  GLOBAL TV *__restrict__ d1 = gl((TV *)D.d1);
  GLOBAL TV *__restrict__ x = gl((TV *)D.x);
  int64_t i0, i1;
  ew_rows(D.n, m.y, D.A.grid, i0, i1);
  for (int64_t i = i0 + threadIdx.x; i < i1; i += kBlock) {
    d0[i] = (TV)0;
    d1[i] = (TV)0;
    if (zero_x) x[i] = (TV)0;
  }
}

// Refinement steps over FP64 system views (A = FP64 copy, x = x64, b = b64,
// r0 = r64; s points at the inner solve's x and t at its right-hand side, both
// in the vector type), with rn = sqrt(st[0].true_rr) of each view:
//   update: x64 += rn * x_inner;   rhs: b_inner = (1 / rn) * r64.
template <typename TV>
__global__ __launch_bounds__(kBlock) void k_outer(const SysDev *__restrict__ dir, const int2 *__restrict__ map,
                                                  int what) {
  const int2 m = map[blockIdx.x];
  const SysDev &D = dir[m.x];
  const double rn = sqrt(gl(D.st)[0].true_rr);
  int64_t i0, i1;
  ew_rows(D.n, m.y, D.A.grid, i0, i1);
  if (what == 0) {
    GLOBAL double *__restrict__ x64 = gl((double *)D.x);
    GLOBAL const TV *__restrict__ c = gl((const TV *)D.s);
    for (int64_t i = i0 + threadIdx.x; i < i1; i += kBlock) x64[i] = x64[i] + rn * (double)c[i];
  } else {
    const double sc = 1.0 / rn;
    GLOBAL const double *__restrict__ r64 = gl((const double *)D.r0);
    GLOBAL TV *__restrict__ bi = gl((TV *)D.t);
    for (int64_t i = i0 + threadIdx.x; i < i1; i += kBlock) bi[i] = (TV)(sc * r64[i]);
  }
}

// One thread per system of the set.
__global__ void k_state_restart(const SysDev *__restrict__ dir, const int32_t *__restrict__ set, int nset) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nset) return;
  GLOBAL State &S = gl(dir[set[k]].st)[0];
  S.done = 0;
  S.status = ST_RUNNING;
  S.alpha = 0.0;
  S.beta = 0.0;
}

template <typename TV>
__global__ __launch_bounds__(kBlock) void k_norm_b(const SysDev *__restrict__ dir, const int2 *__restrict__ map) {
  __shared__ Acc sh[4 * (kBlock / 64)];
  const int2 m = map[blockIdx.x];
  const SysDev &D = dir[m.x];
  GLOBAL const TV *__restrict__ b = gl((const TV *)D.b);
  Acc part[1] = {{0.0, 0.0}};
  // local workgroup l adds the contiguous slice l of b
  const int G = D.gB, l = m.y;
  const int64_t i0 = (int64_t)l * D.n / G, i1 = (int64_t)(l + 1) * D.n / G;
#pragma unroll 4
  for (int64_t i = i0 + threadIdx.x; i < i1; i += kBlock) acc_prod(part[0], b[i], b[i]);
  put_partials<1>(part, gl(D.pb), l, G, sh);
}

// One workgroup per system of the set: ||b||^2 (what = 0, also tol * ||b||
// and the b = 0 test) or ||b - A x||^2 (what = 1) from its partials into st[0].
__global__ __launch_bounds__(kBlock) void k_reduce_state(const SysDev *__restrict__ dir,
                                                         const int32_t *__restrict__ set, int what) {
  __shared__ Acc sh[4 * (kBlock / 64)];
  const SysDev &D = dir[set[blockIdx.x]];
  double v[1];
  if (what == 0)
    sum_partials<1>(gl(D.pb), D.gB, v, sh);
  else
    sum_partials<1>(gl(D.ptr), D.A.grid, v, sh);
  if (threadIdx.x != 0) return;
  GLOBAL State &S = gl(D.st)[0];
  if (what == 0) {
    S.bb = v[0];
    S.tol_nb = S.tol * sqrt(v[0]);
    if (v[0] == 0.0) {
      S.status = ST_ZERO_B;
      S.done = 1;
    }
  } else {
    S.true_rr = v[0];
  }
}

template <typename TS, typename TD>
__global__ void k_convert(const TS *__restrict__ src, TD *__restrict__ dst, int64_t n, double scale) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    dst[i] = (TD)(scale * (double)src[i]);
}

template <typename T>
__global__ void k_fill(T *__restrict__ p, int64_t n, T v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

template <typename TC>
__global__ void k_refine_update(int32_t n, double *__restrict__ x64, const TC *__restrict__ c, double scale) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    x64[i] = x64[i] + scale * (double)c[i];
}

// Streaming probes of the HBM ceiling (and the reference for calibrating the
// memory-traffic counters): 16-byte nontemporal accesses, four per lane in
// flight (all loads of a round issued before its stores), grid-stride rounds.
constexpr int kStreamUnroll = 4;

__global__ __launch_bounds__(kBlock) void k_copy(const u32x4 *__restrict__ src_, u32x4 *__restrict__ dst_, int64_t n16) {
  GLOBAL const u32x4 *src = gl(src_);
  GLOBAL u32x4 *dst = gl(dst_);
  constexpr int U = kStreamUnroll;
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  for (; i + (U - 1) * stride < n16; i += U * stride) {
    u32x4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = __builtin_nontemporal_load(src + i + u * stride);
#pragma unroll
    for (int u = 0; u < U; ++u) __builtin_nontemporal_store(v[u], dst + i + u * stride);
  }
  for (; i < n16; i += stride) __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}

// Read-only stream: the words are folded with xor, and a workgroup writes its
// fold only if it equals a value no test data produces (so the loads stay).
__global__ __launch_bounds__(kBlock) void k_read(const u32x4 *__restrict__ src_, int64_t n16,
                                                 uint32_t *__restrict__ sink_) {
  GLOBAL const u32x4 *src = gl(src_);
  constexpr int U = kStreamUnroll;
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  u32x4 acc = {0u, 0u, 0u, 0u};
  for (; i + (U - 1) * stride < n16; i += U * stride) {
    u32x4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = __builtin_nontemporal_load(src + i + u * stride);
#pragma unroll
    for (int u = 0; u < U; ++u) acc ^= v[u];
  }
  for (; i < n16; i += stride) acc ^= __builtin_nontemporal_load(src + i);
  if (acc.x == 0x9e3779b9u && acc.y == 0x7f4a7c15u && acc.z == 0x85ebca6bu && acc.w == 0xc2b2ae35u)
    gl(sink_)[blockIdx.x] = acc.x;
}

// ------------------------------------------------ FSAI construction on the device

// One wave (the whole workgroup) per row; LDS holds S = A[J,J] (m x m,
// row-major), g (m) and J (m).
__global__ __launch_bounds__(64) void k_fsai_rows(const int32_t *__restrict__ rp_, const int32_t *__restrict__ ci_,
                                                  const double *__restrict__ v_, const int32_t *__restrict__ dpos_,
                                                  const int32_t *__restrict__ lrp_, int32_t n, int32_t mmax,
                                                  double *__restrict__ lv_, int32_t *__restrict__ err_) {
  extern __shared__ double smem[];
  GLOBAL const int32_t *rp = gl(rp_), *ci = gl(ci_), *dpos = gl(dpos_), *lrp = gl(lrp_);
  GLOBAL const double *v = gl(v_);
  GLOBAL double *lv = gl(lv_);
  GLOBAL int32_t *err = gl(err_);
  double *S = smem;
  double *g = smem + (size_t)mmax * mmax;
  int32_t *J = (int32_t *)(g + mmax);
  const int lane = threadIdx.x;
  for (int32_t i = blockIdx.x; i < n; i += gridDim.x) {
    const int32_t r0 = rp[i];
    const int m = dpos[i] - r0 + 1;
    for (int a = lane; a < m; a += 64) J[a] = ci[r0 + a];
    __syncthreads();
    // lower part of S: S[a][b] = A[J[a], J[b]] (b <= a), merging row J[a]'s
    // columns up to its diagonal with J
    for (int a = lane; a < m; a += 64) {
      const int32_t row = J[a];
      int32_t k = rp[row];
      const int32_t kend = dpos[row];
      double *Sa = S + (size_t)a * m;
      int b = 0;
      while (b <= a) {
        if (k > kend) {
          Sa[b++] = 0.0;
          continue;
        }
        const int32_t c = ci[k], jb = J[b];
        if (c == jb) {
          Sa[b++] = v[k++];
        } else if (c < jb) {
          ++k;
        } else {
          Sa[b++] = 0.0;
        }
      }
    }
    __syncthreads();
    // Cholesky, column by column: the pivot by lane 0, the column below it by
    // one lane per entry, each sum left to right
    for (int c = 0; c < m; ++c) {
      if (lane == 0) {
        double dsum = S[(size_t)c * m + c];
        for (int k = 0; k < c; ++k) dsum -= S[(size_t)c * m + k] * S[(size_t)c * m + k];
        if (!(dsum > 0.0)) {
          err[0] = 1;
          dsum = 1.0;
        }
        S[(size_t)c * m + c] = sqrt(dsum);
      }
      __syncthreads();
      const double l = S[(size_t)c * m + c];
      for (int a = c + 1 + lane; a < m; a += 64) {
        double e = S[(size_t)a * m + c];
        for (int k = 0; k < c; ++k) e -= S[(size_t)a * m + k] * S[(size_t)c * m + k];
        S[(size_t)a * m + c] = e / l;
      }
      __syncthreads();
    }
    // back substitution L^T g = e_last
    if (lane == 0) {
      const int32_t base = lrp[i];
      for (int a = m - 1; a >= 0; --a) {
        double e = (a == m - 1) ? 1.0 : 0.0;
        for (int k = a + 1; k < m; ++k) e -= S[(size_t)k * m + a] * g[k];
        g[a] = e / S[(size_t)a * m + a];
        lv[base + a] = g[a];
      }
    }
    __syncthreads();
  }
}

// The same for short rows, one thread per row: S, g and J of each lane
// interleaved in LDS (element e of a lane at e * 64 + lane: no bank
// conflicts), every sum in the same order. A wave per row leaves 60 of 64
// lanes idle on a 4-entry row: 64^3 (262,144 rows of up to 4) 477 -> 35 us.
__global__ __launch_bounds__(64) void k_fsai_short(const int32_t *__restrict__ rp_, const int32_t *__restrict__ ci_,
                                                   const double *__restrict__ v_, const int32_t *__restrict__ dpos_,
                                                   const int32_t *__restrict__ lrp_, int32_t n, int32_t mmax,
                                                   double *__restrict__ lv_, int32_t *__restrict__ err_) {
  extern __shared__ double smem[];
  GLOBAL const int32_t *rp = gl(rp_), *ci = gl(ci_), *dpos = gl(dpos_), *lrp = gl(lrp_);
  GLOBAL const double *v = gl(v_);
  GLOBAL double *lv = gl(lv_);
  const int lane = threadIdx.x;
  double *S = smem + lane, *g = smem + (size_t)mmax * mmax * 64 + lane;
  int32_t *J = (int32_t *)(smem + ((size_t)mmax * mmax + mmax) * 64) + lane;
  for (int64_t i = (int64_t)blockIdx.x * 64 + lane; i < n; i += (int64_t)gridDim.x * 64) {
    const int32_t r0 = rp[i];
    const int m = dpos[i] - r0 + 1;
    for (int a = 0; a < m; ++a) J[a * 64] = ci[r0 + a];
    // lower part of S = A[J,J]: row J[a]'s columns up to its diagonal merged with J
    for (int a = 0; a < m; ++a) {
      const int32_t row = J[a * 64];
      int32_t k = rp[row];
      const int32_t kend = dpos[row];
      for (int b = 0; b <= a; ++b) {
        const int32_t jb = J[b * 64];
        while (k <= kend && ci[k] < jb) ++k;
        S[(a * m + b) * 64] = (k <= kend && ci[k] == jb) ? v[k] : 0.0;
      }
    }
    for (int c = 0; c < m; ++c) {  // Cholesky, column by column, each sum left to right
      double dsum = S[(c * m + c) * 64];
      for (int k = 0; k < c; ++k) dsum -= S[(c * m + k) * 64] * S[(c * m + k) * 64];
      if (!(dsum > 0.0)) {
        gl(err_)[0] = 1;
        dsum = 1.0;
      }
      const double l = sqrt(dsum);
      S[(c * m + c) * 64] = l;
      for (int a = c + 1; a < m; ++a) {
        double e = S[(a * m + c) * 64];
        for (int k = 0; k < c; ++k) e -= S[(a * m + k) * 64] * S[(c * m + k) * 64];
        S[(a * m + c) * 64] = e / l;
      }
    }
    const int32_t base = lrp[i];
    for (int a = m - 1; a >= 0; --a) {  // back substitution L^T g = e_last
      double e = (a == m - 1) ? 1.0 : 0.0;
      for (int k = a + 1; k < m; ++k) e -= S[(k * m + a) * 64] * g[k * 64];
      e = e / S[(a * m + a) * 64];
      g[a * 64] = e;
      lv[base + a] = e;
    }
  }
}

__global__ __launch_bounds__(kBlock) void k_absmax(const double *__restrict__ x, int64_t m, double *__restrict__ part) {
  __shared__ double sh[kBlock / 64];
  double a = 0.0;
  for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < m; k += (int64_t)gridDim.x * kBlock)
    a = fmax(a, fabs(x[k]));
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) a = fmax(a, __shfl_xor(a, off));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = a;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kBlock / 64; ++w) a = fmax(a, sh[w]);
    part[blockIdx.x] = a;
  }
}

// Rounding to nearest even onto a format with `sig` significant bits, least
// normal exponent emin and largest finite value vmax (subnormals included,
// beyond vmax: infinity); every step is exact.
__device__ double round_sig(double v, int sig, int emin, double vmax) {
  if (v == 0.0 || !isfinite(v)) return v;
  int e;
  frexp(fabs(v), &e);
  int q = e - sig;
  if (e - 1 < emin) q = emin - (sig - 1);
  double r = ldexp(rint(ldexp(fabs(v), -q)), q);
  if (r > vmax) r = INFINITY;
  return copysign(r, v);
}

__device__ uint16_t bf16_bits(double v) {
  return (uint16_t)(__float_as_uint((float)round_sig(v, 8, -126, 3.3895313892515355e38)) >> 16);
}

__device__ uint16_t f16_bits(double v) {
  const double r = round_sig(v, 11, -14, 65504.0);
  if (isinf(r)) return r > 0 ? 0x7C00 : 0xFC00;
  if (isnan(r)) return 0x7E00;
  const uint16_t sign = signbit(r) ? 0x8000 : 0;
  const double a = fabs(r);
  if (a == 0.0) return sign;
  int e;
  const double mnt = frexp(a, &e);  // a = mnt 2^e, mnt in [0.5, 1)
  if (e - 1 >= -14) return sign | (uint16_t)((e - 1 + 15) << 10) | (uint16_t)rint((mnt * 2.0 - 1.0) * 1024.0);
  return sign | (uint16_t)rint(a * 16777216.0);  // subnormal: multiples of 2^-24
}

// Store entry idx of `row` (column col) in M's layout: CSR, sliced ELL, or
// sliced diagonals (the slot of offset col - row among the slice's offsets).
__device__ __forceinline__ void store_val(const DevCSR &M, int32_t row, int32_t idx, int32_t col, double x) {
  int64_t p;
  if (M.fmt == FMT_SELL) {
    p = ((int64_t)gl(M.blk)[row / kSliceRows] + idx) * kSliceRows + row % kSliceRows;
  } else if (M.fmt == FMT_SDIA) {
    GLOBAL const int32_t *off = gl(M.ci);
    int32_t lo = gl(M.blk)[row / kSliceRows], hi = gl(M.blk)[row / kSliceRows + 1] - 1;
    const int32_t d = col - row;
    while (lo < hi) {  // the slice lists every offset of its rows, so d is found
      const int32_t mid = lo + (hi - lo) / 2;
      if (off[mid] < d)
        lo = mid + 1;
      else
        hi = mid;
    }
    p = (int64_t)lo * kSliceRows + row % kSliceRows;
  } else {
    p = (int64_t)gl(M.rp)[row] + idx;
  }
  switch (M.dtype) {
    case F64: gl((double *)M.val)[p] = x; break;
    case F32: gl((float *)M.val)[p] = (float)x; break;
    case BF16: gl((uint16_t *)M.val)[p] = bf16_bits(x); break;
    default: gl((uint16_t *)M.val)[p] = f16_bits(x); break;
  }
}

__global__ __launch_bounds__(kBlock) void k_fsai_place(const int32_t *__restrict__ rp_, const int32_t *__restrict__ ci_,
                                                       const int32_t *__restrict__ dpos_,
                                                       const int32_t *__restrict__ lrp_, const double *__restrict__ lv_,
                                                       int32_t n, double scale, DevCSR GT, DevCSR G,
                                                       int32_t *__restrict__ err_) {
  GLOBAL const int32_t *rp = gl(rp_), *ci = gl(ci_), *dpos = gl(dpos_), *lrp = gl(lrp_);
  GLOBAL const double *lv = gl(lv_);
  for (int32_t i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
    const int32_t r0 = rp[i], m = dpos[i] - r0 + 1, base = lrp[i];
    for (int32_t k = 0; k < m; ++k) {
      const int32_t j = ci[r0 + k];
      const double x = lv[base + k] * scale;
      store_val(GT, i, k, j, x);
      // entry (j, i) of G = G_L^T: its rank in the upper part of A's row j
      int32_t lo = dpos[j], hi = rp[j + 1] - 1;
      while (lo < hi) {
        const int32_t mid = lo + (hi - lo) / 2;
        if (ci[mid] < i)
          lo = mid + 1;
        else
          hi = mid;
      }
      if (lo > rp[j + 1] - 1 || ci[lo] != i) {
        gl(err_)[0] = 2;
        continue;
      }
      store_val(G, j, lo - dpos[j], i, x);
    }
  }
}

// The allocation-free entry point's scratch: one copy per device, allocated
// by the runtime with the code object. Host code uses only the per-device
// address that hipGetSymbolAddress returns for it.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t static_scratch(int device, void **ptr) {
  *ptr = nullptr;
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[device]) {
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[device] = p;
  }
  *ptr = g_scratch_ptr[device];
  return hipSuccess;
}

// ---------------------------------------------------------------- launchers

static inline int ew_grid(int64_t n) {
  int64_t g = (n + kBlock - 1) / kBlock;
  if (g > 4096) g = 4096;
  return (int)(g < 1 ? 1 : g);
}

#define PCG_DISPATCH_G(gdt, TG, ...)                          \
  switch (gdt) {                                              \
    case F64: { using TG = double; __VA_ARGS__; break; }      \
    case F32: { using TG = float; __VA_ARGS__; break; }       \
    case BF16: { using TG = bf16_t; __VA_ARGS__; break; }     \
    case F16: { using TG = _Float16; __VA_ARGS__; break; }    \
    default: return hipErrorInvalidValue;                     \
  }

#define PCG_DISPATCH_V(vdt, TV, ...)                          \
  switch (vdt) {                                              \
    case F64: { using TV = double; __VA_ARGS__; break; }      \
    case F32: { using TV = float; __VA_ARGS__; break; }       \
    default: return hipErrorInvalidValue;                     \
  }

// Plain launch, or with events on the dispatch when timing.
#define PCG_LAUNCH(kern, grid, s, e0, e1, ...)                                                  \
  do {                                                                                          \
    if ((e0) || (e1))                                                                           \
      hipExtLaunchKernelGGL(kern, dim3(grid), dim3(kBlock), 0, s, e0, e1, 0, __VA_ARGS__);     \
    else                                                                                        \
      hipLaunchKernelGGL(kern, dim3(grid), dim3(kBlock), 0, s, __VA_ARGS__);                   \
  } while (0)

// A launch over one system passes its record (LaunchSet::one) instead of a map.
#define PCG_ONE(lmap)                                  \
  const SysDev one = L.one ? *L.one : SysDev{};        \
  const int2 *map = L.one ? nullptr : (lmap)

// Whether a single system's product takes the kernels built for one layout: not
// sliced diagonals (the kernels here hold their two-row walk), and not CSR of
// long rows, where a block holds few rows and the threads that sum them bound
// it: at 470 entries per row (72,000 rows) the A-kernel takes 237 us here against
// 255 in FP64 and the G^T-kernel (237 per row) 152 against 167 in FP32. The line
// lies where the two begin to part; below it they stay within 5% of each other in
// each kernel and type (an iteration with G on A's pattern, here and there: 40,000
// rows of 145 137.4 and 140.9 us in FP64, 119.4 and 118.8 in FP32, of 175 159.7 and
// 159.1, 136.4 and 134.5; 72,000 rows of 190 355.8 and 347.9, 284.9 and 286.7), above
// it by up to 9% (72,000 rows of 300: 567.8 and 568.5, 437.4 and 448.9).
static bool one_layout(const DevCSR &M) {
  return M.fmt != FMT_SDIA && !(M.fmt == FMT_CSR && (int64_t)M.nnz > (int64_t)192 * M.n);
}

hipError_t launch_iter_A(const Types &ty, const LaunchSet &L, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  if (L.nA == 0) return hipSuccess;
  if (L.one && one_layout(L.one->A)) return launch_one_A(ty, L, s, e0, e1);
  const bool u4 = L.uw_a == 4;
  PCG_ONE(L.mapA);
  if (ty.vec == F64 && ty.a == F64) {
    if (u4)
      PCG_LAUNCH((k_iter_A<double, double, 4>), L.nA, s, e0, e1, L.dir, map, one);
    else
      PCG_LAUNCH((k_iter_A<double, double, 8>), L.nA, s, e0, e1, L.dir, map, one);
  } else if (ty.vec == F32 && ty.a == F32) {
    if (u4)
      PCG_LAUNCH((k_iter_A<float, float, 4>), L.nA, s, e0, e1, L.dir, map, one);
    else
      PCG_LAUNCH((k_iter_A<float, float, 8>), L.nA, s, e0, e1, L.dir, map, one);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_iter_GT(const Types &ty, const LaunchSet &L, int mode, hipStream_t s, hipEvent_t e0,
                          hipEvent_t e1) {
  if (L.nGT == 0) return hipSuccess;
  if (L.one && one_layout(L.one->GT)) return launch_one_GT(ty, L, mode, s, e0, e1);
  PCG_ONE(L.mapGT);
  PCG_DISPATCH_V(ty.vec, TV, PCG_DISPATCH_G(ty.g, TG, {
    PCG_LAUNCH((k_iter_GT<TV, TG>), L.nGT, s, e0, e1, L.dir, map, one, mode);
  }));
  return hipGetLastError();
}

hipError_t launch_iter_G(const Types &ty, const LaunchSet &L, bool has_eps, int mode, hipStream_t s, hipEvent_t e0,
                         hipEvent_t e1, uint64_t *report) {
  if (L.nG == 0) return hipSuccess;
  if (L.one && one_layout(L.one->G)) return launch_one_G(ty, L, has_eps, mode, s, e0, e1, report);
  PCG_ONE(L.mapG);
  PCG_DISPATCH_V(ty.vec, TV, PCG_DISPATCH_G(ty.g, TG, {
    if (has_eps)
      PCG_LAUNCH((k_iter_G<TV, TG, true>), L.nG, s, e0, e1, L.dir, map, one, mode, report);
    else
      PCG_LAUNCH((k_iter_G<TV, TG, false>), L.nG, s, e0, e1, L.dir, map, one, mode, report);
  }));
  return hipGetLastError();
}

hipError_t launch_resid(const Types &ty, const LaunchSet &L, int slot_sel, bool with_d, bool reduce,
                        bool respect_done, hipStream_t s) {
  if (L.nA == 0) return hipSuccess;
  PCG_ONE(L.mapA);
  if (ty.vec == F64 && ty.a == F64) {
    hipLaunchKernelGGL((k_resid<double, double>), dim3(L.nA), dim3(kBlock), 0, s, L.dir, map, one, slot_sel,
                       (int)with_d, (int)reduce, (int)respect_done);
  } else if (ty.vec == F32 && ty.a == F32) {
    hipLaunchKernelGGL((k_resid<float, float>), dim3(L.nA), dim3(kBlock), 0, s, L.dir, map, one, slot_sel,
                       (int)with_d, (int)reduce, (int)respect_done);
  } else {
    return hipErrorInvalidValue;
  }
  if (reduce) hipLaunchKernelGGL(k_reduce_state, dim3(L.nset), dim3(kBlock), 0, s, L.dir, L.set, 1);
  return hipGetLastError();
}

hipError_t launch_norm_b(const Types &ty, const LaunchSet &L, hipStream_t s) {
  if (L.nB == 0) return hipSuccess;
  PCG_DISPATCH_V(ty.vec, TV, {
    hipLaunchKernelGGL((k_norm_b<TV>), dim3(L.nB), dim3(kBlock), 0, s, L.dir, L.mapB);
  });
  hipLaunchKernelGGL(k_reduce_state, dim3(L.nset), dim3(kBlock), 0, s, L.dir, L.set, 0);
  return hipGetLastError();
}

hipError_t launch_zero_dirs(const Types &ty, const LaunchSet &L, bool zero_x, hipStream_t s) {
  if (L.nA == 0) return hipSuccess;
  PCG_DISPATCH_V(ty.vec, TV, {
    hipLaunchKernelGGL((k_zero_dirs<TV>), dim3(L.nA), dim3(kBlock), 0, s, L.dir, L.mapA, (int)zero_x);
  });
  return hipGetLastError();
}

hipError_t launch_outer(int vec_dtype, const LaunchSet &L64, int what, hipStream_t s) {
  if (L64.nA == 0) return hipSuccess;
  PCG_DISPATCH_V(vec_dtype, TV, {
    hipLaunchKernelGGL((k_outer<TV>), dim3(L64.nA), dim3(kBlock), 0, s, L64.dir, L64.mapA, what);
  });
  return hipGetLastError();
}

hipError_t launch_state_restart(const LaunchSet &L, hipStream_t s) {
  if (L.nset == 0) return hipSuccess;
  hipLaunchKernelGGL(k_state_restart, dim3((L.nset + 255) / 256), dim3(256), 0, s, L.dir, L.set, L.nset);
  return hipGetLastError();
}

hipError_t launch_convert(int src_dtype, const void *src, int dst_dtype, void *dst, int64_t n, double scale,
                          hipStream_t s) {
  PCG_DISPATCH_V(src_dtype, TS, PCG_DISPATCH_V(dst_dtype, TD, {
    hipLaunchKernelGGL((k_convert<TS, TD>), dim3(ew_grid(n)), dim3(kBlock), 0, s, (const TS *)src, (TD *)dst, n,
                       scale);
  }));
  return hipGetLastError();
}

hipError_t launch_fill(int dtype, void *p, int64_t n, double value, hipStream_t s) {
  PCG_DISPATCH_V(dtype, TV, {
    hipLaunchKernelGGL((k_fill<TV>), dim3(ew_grid(n)), dim3(kBlock), 0, s, (TV *)p, n, (TV)value);
  });
  return hipGetLastError();
}

hipError_t launch_refine_update(int32_t n, double *x64, const void *c, int c_dtype, double scale, hipStream_t s) {
  PCG_DISPATCH_V(c_dtype, TC, {
    hipLaunchKernelGGL((k_refine_update<TC>), dim3(ew_grid(n)), dim3(kBlock), 0, s, n, x64, (const TC *)c, scale);
  });
  return hipGetLastError();
}

hipError_t launch_fsai_rows(const int32_t *rp, const int32_t *ci, const double *v, const int32_t *dpos,
                            const int32_t *lrp, int32_t n, int32_t mmax, double *lv, int32_t *err, int grid,
                            hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (mmax < 1 || mmax > kFsaiMaxRow) return hipErrorInvalidValue;
  if (mmax <= kFsaiShortRow) {
    const size_t lds = 64 * (sizeof(double) * ((size_t)mmax * mmax + mmax) + sizeof(int32_t) * mmax);
    const int wgs = (int)std::min<int64_t>(((int64_t)n + 63) / 64, grid);
    hipLaunchKernelGGL(k_fsai_short, dim3(wgs), dim3(64), lds, s, rp, ci, v, dpos, lrp, n, mmax, lv, err);
    return hipGetLastError();
  }
  const size_t lds = sizeof(double) * ((size_t)mmax * mmax + mmax) + sizeof(int32_t) * mmax;
  hipLaunchKernelGGL(k_fsai_rows, dim3(grid), dim3(64), lds, s, rp, ci, v, dpos, lrp, n, mmax, lv, err);
  return hipGetLastError();
}

hipError_t launch_absmax(const double *x, int64_t m, double *part, hipStream_t s) {
  hipLaunchKernelGGL(k_absmax, dim3(kAbsmaxGrid), dim3(kBlock), 0, s, x, m, part);
  return hipGetLastError();
}

hipError_t launch_fsai_place(const int32_t *rp, const int32_t *ci, const int32_t *dpos, const int32_t *lrp,
                             const double *lv, int32_t n, double scale, const DevCSR &GT, const DevCSR &G,
                             int32_t *err, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fsai_place, dim3(ew_grid(n)), dim3(kBlock), 0, s, rp, ci, dpos, lrp, lv, n, scale, GT, G, err);
  return hipGetLastError();
}

hipError_t launch_copy(const void *src, void *dst, int64_t bytes, int grid, hipStream_t s) {
  hipLaunchKernelGGL(k_copy, dim3(grid), dim3(kBlock), 0, s, (const u32x4 *)src, (u32x4 *)dst, bytes / 16);
  return hipGetLastError();
}

hipError_t launch_read(const void *src, int64_t bytes, uint32_t *sink, int grid, hipStream_t s) {
  hipLaunchKernelGGL(k_read, dim3(grid), dim3(kBlock), 0, s, (const u32x4 *)src, bytes / 16, sink);
  return hipGetLastError();
}

}  // namespace pcgk
