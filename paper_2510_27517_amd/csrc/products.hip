// Products with one stored matrix outside the iteration: y = M x, and the
// multi-probe products and sums of the preconditioner losses. Each row is
// summed left to right in CSR order, in every layout.
// Built with floating-point contraction off, like every kernel here.
#include <hip/hip_runtime.h>
#include <algorithm>
#include <cstdint>

#include "device.h"
#include "kernels.h"

namespace pcgk {

// y[row] = (TY) v, v = the row's sum in TV, or a sum + b z[row] with AXPY; x, y
// and z in FP64 or TV: the caller's FP64 vectors are read and written in
// place, converted as they are gathered, with no copies around the product.
// FMT: sliced diagonals have kernels of their own; built with the others, a change
// to the staging of CSR blocks slowed their nontemporal walk (128^3, G x: 29.3 ->
// 32.5 us).
template <typename TV, typename TM, typename TX, typename TY, bool AXPY, int FMT>
__global__ __launch_bounds__(kBlock) PCG_OCCUPANCY void k_spmv(DevCSR Md, const TX *__restrict__ x_,
                                                              TY *__restrict__ y_, TV a, TV b,
                                                              const double *__restrict__ z_) {
  __shared__ TV lds[kLdsBytes / sizeof(TV)];
  const Mat<TM> M = mat<TM, FMT>(Md);
  GLOBAL const TX *__restrict__ x = gl(x_);
  GLOBAL TY *__restrict__ y = gl(y_);
  GLOBAL const double *z = gl(z_);
  for_rows<TV, 8, 8>(
      M, blockIdx.x, gridDim.x, lds,
      [&](int row) { return RowVals<TV>{AXPY ? (TV)z[row] : (TV)0, (TV)0, (TV)0}; },
      [&](int j) -> TV { return (TV)x[j]; },
      [&](int row, TV sum, const RowVals<TV> &pv) { y[row] = (TY)(AXPY ? a * sum + b * pv.a : sum); });
}

template <typename TM>
__device__ __forceinline__ double ld64(GLOBAL const TM *p, int64_t k) {
  return (double)ldval<false>(p, k);
}

// What each of the losses' five sums adds for one entry (w, y) of a probe.
__device__ __forceinline__ void loss_terms(double (&acc)[5], double w, double y, double na) {
  const double e = y / na - w, f = y - w;
  acc[0] += e * e;
  acc[1] += f * f;
  acc[2] += w * y;
  acc[3] += y * y;
  acc[4] += w * w;
}

// Y = c (M X) + d Z for k probes, n x k row-major; LOSS: Y is not stored, its
// terms of the losses against Z = W are summed instead.
//
// LPR lanes per row and PV probes per lane (two make every access 16 bytes): a
// wave works on 64 / LPR adjacent rows of one slice. The product is bound by
// the n x k vectors: each die takes a contiguous eighth of the rows, its
// workgroups interleaved, so that the rows gathered again by later ones (the
// far diagonals' by the next plane) come from that die's L2; Y is stored past
// the caches, which keeps the window of X there. At 96^3 with 32 probes the
// G^T- and G-products take 120 us (counters: 541 MB read and written, 1.13 of
// the least, at the copy kernel's 4.8 TB/s) and A's 168 (929 MB read, 1.8 of
// the least: with diagonals on both sides the window of U outgrows the L2; in
// halves of 16 probes it took 180). All three and the probes' copy and the
// separate pass over W and Y took 1240 us before. Two entries in flight per
// lane: with four, the waves drift further apart and A's product re-reads
// more (202 us), with eight 278. Over one probe per lane four: those are the
// launches of few waves or of an odd count, where latency binds (20,000 rows of
// 100, 7 probes: 0.90 of the time with two). 3x3 blocks go a block at a time in
// kernels of their own (BSR), with one index and no division per entry (elasticity 24^3, 32 probes: 233 -> 170
// us). thin: a loss launch with little more than one turn of rows per wave gives
// a workgroup's waves rows apart, so that no CU takes two full workgroups while
// others have one (elasticity 8^3, 8 probes: 66 -> 52 us).
template <typename TM, int LPR, int PV, int NT, bool LOSS, bool BSR>
__device__ __forceinline__ void spmm(const DevCSR &Md, int32_t k, GLOBAL const double *X, int32_t ldx, double c,
                                     GLOBAL const double *Z, int32_t ldz, double d, GLOBAL double *Y, int32_t ldy,
                                     double na, GLOBAL double *part, int32_t ldp, double *sh) {
  const Mat<TM> M = mat<TM, BSR ? FMT_BSR3 : -1>(Md);
  constexpr int RPW = 64 / LPR, NW = NT / 64, CH = LPR * PV;
  const int lane = threadIdx.x & 63, grp = lane / LPR, pl = (lane % LPR) * PV;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l = blockIdx.x, W = gridDim.x >> 3, die = l & 7, w = l >> 3;
  const int T = (M.n + RPW - 1) / RPW;
  const bool thin = LOSS && T < 2 * (int)gridDim.x * NW;
  const int t0 = (int)((int64_t)die * T / 8), t1 = (int)((int64_t)(die + 1) * T / 8);
  for (int32_t p0 = 0; p0 < k; p0 += CH) {
    const int32_t p = p0 + pl;
    const bool pact = p < k;  // PV = 2 only for even k: both probes exist or neither
    double acc[LOSS ? PV : 1][5] = {};
    for (int t = t0 + (thin ? wv * W + w : w * NW + wv); t < t1; t += W * NW) {
      const int32_t base = t * RPW, row = min(base + grp, M.n - 1);
      const bool act = pact && base + grp < M.n;
      double sum[PV] = {};
      // N entries in CSR order with all their loads in flight; past the row's end
      // they repeat its last entry (in bounds) and are not added
      auto batch = [&](int e, int len, auto width, auto entry) {
        constexpr int N = decltype(width)::value;
        double a[N], x[N][PV];
#pragma unroll
        for (int u = 0; u < N; ++u) {
          const int ee = min(e + u, len - 1);
          int32_t col;
          entry(ee, col, a[u]);
          const int64_t at = (int64_t)col * ldx + (pact ? p : 0);
          if constexpr (PV == 2) {
            const Pair<double> v = ld_pair(X, at);
            x[u][0] = v.x;
            x[u][1] = v.y;
          } else {
            x[u][0] = X[at];
          }
        }
#pragma unroll
        for (int u = 0; u < N; ++u)
          if (e + u < len)
#pragma unroll
            for (int j = 0; j < PV; ++j) sum[j] += a[u] * x[u][j];
      };
      auto walk = [&](int len, auto entry) {
        int e = 0;
        if constexpr (PV == 1)
          for (; e + 4 <= len; e += 4) batch(e, len, std::integral_constant<int, 4>{}, entry);
        for (; e < len; e += 2) batch(e, len, std::integral_constant<int, 2>{}, entry);
      };
      if (!BSR && M.fmt == FMT_SDIA) {  // one offset per slice entry; stored zeros add +0
        const int sl = __builtin_amdgcn_readfirstlane(min(base, M.n - 1) / kSliceRows);
        const int o0 = ro(M.blk)[sl], wd = ro(M.blk)[sl + 1] - o0;
        GLOBAL const TM *vv = M.val + (int64_t)o0 * kSliceRows + row % kSliceRows;
        walk(wd, [&](int e, int32_t &col, double &a) {
          col = min(max(row + ro(M.ci)[o0 + e], 0), M.n - 1);
          a = ld64(vv, (int64_t)e * kSliceRows);
        });
      } else if (BSR) {  // a block at a time: three entries of the row
        const int32_t R = row / 3, sub = row % 3, sl = R / kBSliceRows, rr = R % kBSliceRows;
        const int32_t o0 = M.blk[sl], wd = M.blk[sl + 1] - o0;
        GLOBAL const int32_t *bc = M.ci + (int64_t)o0 * kBSliceRows + rr;
        GLOBAL const TM *bv = M.val + (int64_t)o0 * (9 * kBSliceRows) +
                              (sizeof(TM) == 8 ? sub * kBSliceRows + rr : 9 * rr + 3 * sub);
        for (int b = 0; b < wd; ++b, bc += kBSliceRows, bv += 9 * kBSliceRows) {
          const int32_t c0 = 3 * *bc;
          auto entry = [&](int j, int32_t &col, double &a) {
            col = c0 + j;
            a = ld64(bv, sizeof(TM) == 8 ? 3 * kBSliceRows * j : j);
          };
          if constexpr (LOSS && PV == 2) {  // three at once would spill
            batch(0, 3, std::integral_constant<int, 2>{}, entry);
            batch(2, 3, std::integral_constant<int, 1>{}, entry);
          } else {
            batch(0, 3, std::integral_constant<int, 3>{}, entry);
          }
        }
      } else if (M.fmt == FMT_SELL) {  // padded entries add +0 (value 0, valid column)
        const int sl = __builtin_amdgcn_readfirstlane(min(base, M.n - 1) / kSliceRows);
        const int o0 = ro(M.blk)[sl], wd = ro(M.blk)[sl + 1] - o0;
        const int64_t q0 = (int64_t)o0 * kSliceRows + row % kSliceRows;
        if (M.idx16)
          walk(wd, [&](int e, int32_t &col, double &a) {
            const int64_t q = q0 + (int64_t)e * kSliceRows;
            col = row + (int32_t)((GLOBAL const int16_t *)M.ci)[q];
            a = ld64(M.val, q);
          });
        else
          walk(wd, [&](int e, int32_t &col, double &a) {
            const int64_t q = q0 + (int64_t)e * kSliceRows;
            col = M.ci[q];
            a = ld64(M.val, q);
          });
      } else {
        const int32_t q0 = M.rp[row], len = M.rp[row + 1] - q0;
        walk(len, [&](int e, int32_t &col, double &a) {
          col = M.ci[q0 + e];
          a = ld64(M.val, q0 + e);
        });
      }
      if (!act) continue;
      const int64_t az = (int64_t)row * ldz + p, at = (int64_t)row * ldy + p;
#pragma unroll
      for (int j = 0; j < PV; ++j) {
        double y = c * sum[j];
        if constexpr (LOSS) {
          loss_terms(acc[j], Z[az + j], y, na);
        } else {
          if (Z) y = y + d * Z[az + j];
          sum[j] = y;
        }
      }
      if constexpr (!LOSS) {
        if constexpr (PV == 2)
          {
            typedef double VW __attribute__((ext_vector_type(2), aligned(8)));
            VW vw;
            vw.x = sum[0];
            vw.y = sum[1];
            __builtin_nontemporal_store(vw, (GLOBAL VW *)(Y + at));
          }
        else
          Y[at] = sum[0];
      }
    }
    if constexpr (LOSS) {
      // the wave's rows of one probe, then the waves in order
#pragma unroll
      for (int q = 0; q < 5; ++q) {
#pragma unroll
        for (int j = 0; j < PV; ++j) {
          double v = acc[j][q];
#pragma unroll
          for (int o = LPR; o < 64; o *= 2) v += __shfl_xor(v, o);
          if (grp == 0) sh[wv * CH + pl + j] = v;
        }
        __syncthreads();
        const int t = threadIdx.x;
        if (t < CH && p0 + t < k) {
          double v = 0.0;
          for (int u = 0; u < NW; ++u) v += sh[u * CH + t];
          part[((int64_t)blockIdx.x * 5 + q) * ldp + p0 + t] = v;
        }
        __syncthreads();
      }
    }
  }
}

template <typename TM, int LPR, int PV, bool BSR>
__global__ __launch_bounds__(kBlock) PCG_OCCUPANCY void k_spmm(DevCSR M, int32_t k, const double *X, int32_t ldx, double c,
                                                              const double *Z, int32_t ldz, double d, double *Y,
                                                              int32_t ldy) {
  spmm<TM, LPR, PV, kBlock, false, BSR>(M, k, gl(X), ldx, c, Z ? gl(Z) : nullptr, ldz, d, gl(Y), ldy, 1.0, nullptr, 0,
                                   nullptr);
}

// The last product of the losses with their sums over its rows: part[(b 5 +
// q) k + p] for workgroup b < kLossGrid (two large workgroups per CU, so that
// the partial sums stay few while every wave slot is taken).
constexpr int kLossThreads = 1024;
template <typename TM, int LPR, int PV, bool BSR>
__global__ __launch_bounds__(kLossThreads) PCG_OCCUPANCY void k_spmm_loss(DevCSR M, int32_t k, const double *X,
                                                                         int32_t ldx, const double *W, int32_t ldw,
                                                                         double na, double *part, int32_t ldp) {
  __shared__ double sh[kLossThreads / 64 * LPR * PV];
  spmm<TM, LPR, PV, kLossThreads, true, BSR>(M, k, gl(X), ldx, 1.0, gl(W), ldw, 0.0, nullptr, 0, na, gl(part), ldp, sh);
}

// One wave per probe: the workgroups' partial sums, each lane's in ascending
// order, then across the lanes, and the three losses.
__global__ __launch_bounds__(64) void k_loss_final(int32_t k, const double *__restrict__ part_,
                                                   double *__restrict__ out_) {
  GLOBAL const double *part = gl(part_);
  GLOBAL double *out = gl(out_);
  for (int32_t p = blockIdx.x; p < k; p += gridDim.x) {
    double q[5] = {0, 0, 0, 0, 0};
#pragma unroll
    for (int b = threadIdx.x; b < kLossGrid; b += 64)
#pragma unroll
      for (int j = 0; j < 5; ++j) q[j] += part[((int64_t)b * 5 + j) * k + p];
#pragma unroll
    for (int o = 1; o < 64; o *= 2)
#pragma unroll
      for (int j = 0; j < 5; ++j) q[j] += __shfl_xor(q[j], o);
    if (threadIdx.x == 0) {
      out[p] = q[0];
      out[(int64_t)k + p] = q[1];
      out[2 * (int64_t)k + p] = q[2] / (sqrt(q[4]) * sqrt(q[3]));
    }
  }
}

// ---------------------------------------------------------------- launchers

#define PCG_PROD_M(dt, TM, ...)                            \
  switch (dt) {                                            \
    case F64: { using TM = double; __VA_ARGS__; break; }   \
    case F32: { using TM = float; __VA_ARGS__; break; }    \
    case BF16: { using TM = bf16_t; __VA_ARGS__; break; }  \
    case F16: { using TM = _Float16; __VA_ARGS__; break; } \
    default: return hipErrorInvalidValue;                  \
  }

template <typename TV, typename TM, typename TX, typename TY, int FMT>
static void launch_product_as(const DevCSR &M, const void *x, void *y, const double *z, double a, double b,
                              hipStream_t s) {
  if (z)
    hipLaunchKernelGGL((k_spmv<TV, TM, TX, TY, true, FMT>), dim3(M.grid), dim3(kBlock), 0, s, M, (const TX *)x, (TY *)y,
                       (TV)a, (TV)b, z);
  else
    hipLaunchKernelGGL((k_spmv<TV, TM, TX, TY, false, FMT>), dim3(M.grid), dim3(kBlock), 0, s, M, (const TX *)x,
                       (TY *)y, (TV)0, (TV)0, z);
}

template <typename TV, typename TM, typename TX, typename TY>
static hipError_t launch_product(const DevCSR &M, const void *x, void *y, const double *z, double a, double b,
                                 hipStream_t s) {
  if (M.fmt == FMT_SDIA)
    launch_product_as<TV, TM, TX, TY, FMT_SDIA>(M, x, y, z, a, b, s);
  else
    launch_product_as<TV, TM, TX, TY, -1>(M, x, y, z, a, b, s);
  return hipGetLastError();
}

hipError_t launch_spmv(const Types &ty, const DevCSR &M, int x_dtype, const void *x, int y_dtype, void *y,
                       const double *z, double a, double b, hipStream_t s) {
  if (ty.vec == F64) {
    if (x_dtype != F64 || y_dtype != F64) return hipErrorInvalidValue;
    PCG_PROD_M(M.dtype, TM, return launch_product<double, TM, double, double>(M, x, y, z, a, b, s));
  } else {
    if (M.dtype == F64) return hipErrorInvalidValue;
    PCG_PROD_M(M.dtype, TM, {
      if constexpr (!std::is_same_v<TM, double>) {
        if (x_dtype == F64)
          return y_dtype == F64 ? launch_product<float, TM, double, double>(M, x, y, z, a, b, s)
                                : launch_product<float, TM, double, float>(M, x, y, z, a, b, s);
        if (y_dtype == F64) return launch_product<float, TM, float, double>(M, x, y, z, a, b, s);
      }
    });
  }
  return hipErrorInvalidValue;
}

// The smallest lane groups that hold the probes, two probes per lane where they
// pair up. That halves the accesses but also the waves, so it needs 4,096 of them
// left, half of what the chip holds (losses over 8 probes, paired against one per
// lane: elasticity 36^3, 8,748 waves, 161 and 232 us; 20,000 rows of 100, 1,250
// waves, 216 and 112; elasticity 8^3, 96 waves, 74 and 51; P P^T of 18,000 over 16,
// 2,250 waves, 141 and 108), and more than two probes, which would leave every other
// lane idle (100^3: 91 and 77). Above 64 probes, where a row takes a whole wave
// either way, they pair up always (60^2, 100 probes: 47 and 52).
static void spmm_shape(int32_t n, int32_t k, int &lpr, bool &pair) {
  auto fit = [](int32_t m) {
    int l = 2;
    while (l < m && l < 64) l *= 2;
    return l;
  };
  pair = k > 2 && k % 2 == 0 && (k > 64 || (int64_t)n * fit(k / 2) / 64 >= 4096);
  lpr = fit(pair ? k / 2 : k);
}

#define PCG_SPMM_LPR(lpr_, LPR, ...)                            \
  switch (lpr_) {                                               \
    case 2: { constexpr int LPR = 2; __VA_ARGS__; break; }      \
    case 4: { constexpr int LPR = 4; __VA_ARGS__; break; }      \
    case 8: { constexpr int LPR = 8; __VA_ARGS__; break; }      \
    case 16: { constexpr int LPR = 16; __VA_ARGS__; break; }    \
    case 32: { constexpr int LPR = 32; __VA_ARGS__; break; }    \
    default: { constexpr int LPR = 64; __VA_ARGS__; break; }    \
  }
#define PCG_SPMM_SHAPE(n, k, LPR, PV, ...)           \
  do {                                               \
    int lpr_;                                        \
    bool pair_;                                      \
    spmm_shape(n, k, lpr_, pair_);                   \
    if (pair_) {                                     \
      constexpr int PV = 2;                          \
      PCG_SPMM_LPR(lpr_, LPR, __VA_ARGS__)           \
    } else {                                         \
      constexpr int PV = 1;                          \
      PCG_SPMM_LPR(lpr_, LPR, __VA_ARGS__)           \
    }                                                \
  } while (0)

// A multiple of 8 workgroups, enough to take every row, at most `most`.
static int spmm_grid(int32_t n, int rows_per_wg, int most) {
  const int64_t t = ((int64_t)n + rows_per_wg - 1) / rows_per_wg;
  return (int)std::min<int64_t>((t + 7) / 8 * 8, most);
}

hipError_t launch_spmm(const DevCSR &M, int32_t k, const double *X, int32_t ldx, double c, const double *Z,
                       int32_t ldz, double d, double *Y, int32_t ldy, hipStream_t s) {
  if (M.n <= 0 || k <= 0) return hipSuccess;
  PCG_PROD_M(M.dtype, TM, PCG_SPMM_SHAPE(M.n, k, LPR, PV, {
    const int grid = spmm_grid(M.n, kBlock / LPR, kSpmmGrid);
    if (M.fmt == FMT_BSR3)
      hipLaunchKernelGGL((k_spmm<TM, LPR, PV, true>), dim3(grid), dim3(kBlock), 0, s, M, k, X, ldx, c, Z, ldz, d, Y,
                         ldy);
    else
      hipLaunchKernelGGL((k_spmm<TM, LPR, PV, false>), dim3(grid), dim3(kBlock), 0, s, M, k, X, ldx, c, Z, ldz, d, Y,
                         ldy);
  }));
  return hipGetLastError();
}

hipError_t launch_spmm_loss(const DevCSR &M, int32_t k, const double *X, int32_t ldx, const double *W, int32_t ldw,
                            double na, double *part, int32_t ldp, hipStream_t s) {
  if (M.n <= 0 || k <= 0) return hipSuccess;
#define PCG_LOSS(TM)                                                                                              \
  PCG_SPMM_SHAPE(M.n, k, LPR, PV, {                                                                               \
    if (M.fmt == FMT_BSR3)                                                                                        \
      hipLaunchKernelGGL((k_spmm_loss<TM, LPR, PV, true>), dim3(kLossGrid), dim3(kLossThreads), 0, s, M, k, X, ldx, \
                         W, ldw, na, part, ldp);                                                                  \
    else                                                                                                          \
      hipLaunchKernelGGL((k_spmm_loss<TM, LPR, PV, false>), dim3(kLossGrid), dim3(kLossThreads), 0, s, M, k, X,    \
                         ldx, W, ldw, na, part, ldp);                                                             \
  })
  if (M.dtype == F64)
    PCG_LOSS(double);
  else if (M.dtype == F32)
    PCG_LOSS(float);
  else
    return hipErrorInvalidValue;
#undef PCG_LOSS
  return hipGetLastError();
}

hipError_t launch_loss_final(int32_t k, const double *part, double *out, hipStream_t s) {
  if (k <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_loss_final, dim3(std::min(k, 65536)), dim3(64), 0, s, k, part, out);
  return hipGetLastError();
}

}  // namespace pcgk
