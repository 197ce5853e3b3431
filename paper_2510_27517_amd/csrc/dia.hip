// Iteration kernels over stencil storage (DiaOp): the three launches of one CG
// iteration of a single system whose A and G^T have a few diagonals each.
//
// A stencil matrix in the general layouts is read through slice pointers and
// per-slice offset lists, A with both triangles and G beside G^T. Here one
// lower triangle serves twice: A is symmetric, so entry (r, r + o) is read as
// the stored (r + o, r), and G is G^T's transpose, read the same way. That
// halves A's bytes, lets G's values come from the memory-side cache where the
// G^T-kernel just left them, and needs no metadata: every address of a row
// follows from its number, so a tile's loads are all issued at once.
//
// Rows are summed left to right in column order from zero, as in every other
// layout, and inner products do not depend on how they are split (up to the
// bound in device.h), so a solve has the same bits as through the general kernels. (Diagonal entries that a row does not have are
// stored zeros: each adds +0 to a sum that can never be -0.)
//
// Built with floating-point contraction off, like every kernel here.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <cstdint>

#include "device.h"
#include "kernels.h"

namespace pcgk {

namespace {

// R adjacent entries of a vector or value stream, at any element alignment.
template <typename T, int R>
struct Vec {
  T v[R];
};

template <typename T>
struct Raw {
  using type = T;
};
template <>
struct Raw<bf16_t> {
  using type = uint16_t;
};

template <typename TV, typename TM>
__device__ __forceinline__ TV from_raw(typename Raw<TM>::type u) {
  if constexpr (std::is_same_v<TM, bf16_t>)
    return (TV)__uint_as_float((uint32_t)u << 16);
  else if constexpr (std::is_same_v<TM, _Float16>)
    return (TV)(float)u;
  else
    return (TV)u;
}

// Values [i, i + R) of a stream, converted to the vector type; NT as ldstream.
template <typename TV, int R, bool NT, typename TM>
__device__ __forceinline__ Vec<TV, R> ld_values(GLOBAL const TM *p, int64_t i) {
  using U = typename Raw<TM>::type;
  Vec<TV, R> o;
  if constexpr (R == 1) {
    o.v[0] = from_raw<TV, TM>(ldstream<NT>((GLOBAL const U *)p, i));
  } else {
    typedef U VU __attribute__((ext_vector_type(R), aligned(sizeof(U))));
    GLOBAL const VU *q = (GLOBAL const VU *)((GLOBAL const U *)p + i);
    VU u;
    if constexpr (NT)
      u = __builtin_nontemporal_load(q);
    else
      u = *q;
#pragma unroll
    for (int k = 0; k < R; ++k) o.v[k] = from_raw<TV, TM>(u[k]);
  }
  return o;
}

// Entries [j, j + R) of a vector; CLAMP: each index clamped into [0, n).
template <int R, bool CLAMP, typename TV>
__device__ __forceinline__ Vec<TV, R> ld_vec(GLOBAL const TV *x, int32_t j, int32_t n) {
  Vec<TV, R> o;
  if constexpr (CLAMP) {
#pragma unroll
    for (int k = 0; k < R; ++k) o.v[k] = x[min(max(j + k, 0), n - 1)];
  } else {
    __builtin_memcpy(&o, x + j, sizeof(o));
  }
  return o;
}

// Store entries [j, j + R), those below n when CLAMP.
template <int R, bool CLAMP, typename TV>
__device__ __forceinline__ void st_vec(GLOBAL TV *x, int32_t j, int32_t n, const Vec<TV, R> &v) {
  if constexpr (CLAMP) {
#pragma unroll
    for (int k = 0; k < R; ++k)
      if (j + k < n) x[j + k] = v.v[k];
  } else {
    __builtin_memcpy(x + j, &v, sizeof(v));
  }
}

template <typename TV, int R>
__device__ __forceinline__ void add_terms(Vec<TV, R> &s, const Vec<TV, R> &a, const Vec<TV, R> &x) {
#pragma unroll
  for (int k = 0; k < R; ++k) s.v[k] += a.v[k] * x.v[k];
}

// This workgroup's tiles (64 R consecutive rows, one per wave at a time): each
// die takes a contiguous eighth of them, its workgroups and their waves
// interleaved, so that a die works on one window of rows at any moment and
// small systems spread over all workgroups.
struct Tiles {
  int base, count, first, stride;
};
template <int R>
__device__ __forceinline__ Tiles tiles_of(int n, int l, int grid) {
  constexpr int NW = kBlock / 64;
  const int T = (n + 64 * R - 1) / (64 * R);
  const int W = grid >> 3, x = l & 7, w = l >> 3;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int t0 = (int)((int64_t)x * T / 8), t1 = (int)((int64_t)(x + 1) * T / 8);
  return Tiles{t0, t1 - t0, w + wv * W, W * NW};
}

// A tile lies inside the matrix when no operand index of its rows leaves
// [0, n) (the same for the whole wave).
template <int R>
__device__ __forceinline__ bool inside(int tile, int far, int n) {
  const int a = tile * 64 * R;
  return a >= far && a + 64 * R + far <= n;
}

}  // namespace

// q = A d, partials of d^T q. Each stored diagonal is read at row r (lower
// triangle) and at row r + dist (upper); the second read of a value comes
// dist rows later from L2, which holds the window a die works on. At 128^3
// FP64 (100.7 MB instead of 151.5): 22.5 -> 16.4 us.
template <typename TV, typename TA, int ND, int R, bool NT>
__global__ __launch_bounds__(kBlock) PCG_GT_OCCUPANCY void k_dia_A(DiaOp A, DiaVecs v, int par, int grid) {
  __shared__ Acc sh[4 * (kBlock / 64)];
  const int l = blockIdx.x, n = v.n, lane = threadIdx.x & 63;
  GLOBAL const State &S = gl(v.st)[0];
  GLOBAL TV *__restrict__ q = gl((TV *)v.q);
  GLOBAL const TV *__restrict__ d = gl((const TV *)(par ? v.d1 : v.d0));
  GLOBAL const TA *val = gl((const TA *)A.val);
  const Tiles tl = tiles_of<R>(n, l, grid);
  Acc part[1] = {{0.0, 0.0}};
  bool live = true;
  auto tile = [&](int t, auto first, auto clamp) {
    constexpr bool C = decltype(clamp)::value;
    const int r0 = t * 64 * R + lane * R;
    Vec<TV, R> al[ND], au[ND], xl[ND], xu[ND];
#pragma unroll
    for (int k = ND - 1; k >= 0; --k) {
      al[k] = ld_values<TV, R, NT>(val + k * A.ld, r0);
      xl[k] = ld_vec<R, C>(d, r0 - A.dist[k], n);
    }
#pragma unroll
    for (int k = 1; k < ND; ++k) {
      au[k] = ld_values<TV, R, NT>(val + k * A.ld, r0 + A.dist[k]);
      xu[k] = ld_vec<R, C>(d, r0 + A.dist[k], n);
    }
    if constexpr (decltype(first)::value) {
      live = !S.done;
      if (!live) return;
    }
    Vec<TV, R> s{};
#pragma unroll
    for (int k = ND - 1; k >= 0; --k) add_terms(s, al[k], xl[k]);
#pragma unroll
    for (int k = 1; k < ND; ++k) add_terms(s, au[k], xu[k]);
    st_vec<R, C>(q, r0, n, s);
#pragma unroll
    for (int i = 0; i < R; ++i)
      if (!C || r0 + i < n) acc_prod(part[0], xl[0].v[i], s.v[i]);
  };
  auto any = [&](int t, auto first) {
    if (inside<R>(t, A.dist[ND - 1], n))
      tile(t, first, std::false_type{});
    else
      tile(t, first, std::true_type{});
  };
  int k = tl.first;
  if (k < tl.count)
    any(tl.base + k, std::true_type{});
  else
    live = !S.done;
  if (!live) return;
  for (k += tl.stride; k < tl.count; k += tl.stride) any(tl.base + k, std::false_type{});
  put_partials<1>(part, gl(v.pg), part_slot(l, grid), grid, sh);
}

// alpha; r_{i+1} = r_i - alpha q; t = G^T r_{i+1}; partials of ||r||^2 and
// ||t||^2. The first tile's loads are in flight while alpha is reduced. Tiles
// are taken from the top of the die's range down, as the general kernel does.
// At 128^3 FP64 (134 MB): 25.9 -> 21.2 us, the rest of the gain over the
// general kernel being the metadata and per-slice work it no longer does.
template <typename TV, typename TG, int ND, int R, bool NT>
__global__ __launch_bounds__(kBlock) PCG_GT_OCCUPANCY void k_dia_GT(DiaOp B, DiaVecs v, int par, int gridA,
                                                                    int grid) {
  __shared__ Acc sh[4 * (kBlock / 64)];
  const int l = blockIdx.x, n = v.n, lane = threadIdx.x & 63;
  GLOBAL State *st = gl(v.st);
  GLOBAL const State &S = st[0];
  Acc g[1];
  load_partials<1>(gl(v.pg), gridA, g);
  GLOBAL const TV *__restrict__ q = gl((const TV *)v.q);
  GLOBAL TV *__restrict__ t = gl((TV *)v.t);
  GLOBAL const TV *__restrict__ src = gl((const TV *)(par ? v.r1 : v.r0));
  GLOBAL TV *__restrict__ dst = gl((TV *)(par ? v.r0 : v.r1));
  GLOBAL const TG *val = gl((const TG *)B.val);
  const Tiles tl = tiles_of<R>(n, l, grid);
  double alpha = 0.0, gamma = 0.0;
  TV al = (TV)0;
  bool was_done = false, brk = false;
  auto step = [&]() -> bool {
    if (S.done) {  // stopped earlier: st[1] mirrors st[0]
      was_done = true;
      return false;
    }
    double gv[1];
    reduce_partials<1>(g, gv, sh);
    gamma = gv[0];
    brk = !(gamma > 0.0) || !isfinite(gamma);
    alpha = brk ? 0.0 : S.delta / gamma;  // on breakdown x already holds x_i
    al = (TV)alpha;
    return !brk;
  };
  Acc part[2] = {{0.0, 0.0}, {0.0, 0.0}};
  auto tile = [&](int k, auto first, auto clamp) -> bool {
    constexpr bool C = decltype(clamp)::value;
    const int r0 = (tl.base + tl.count - 1 - k) * 64 * R + lane * R;
    Vec<TV, R> b[ND], s[ND], y[ND];
#pragma unroll
    for (int k2 = ND - 1; k2 >= 0; --k2) {
      s[k2] = ld_vec<R, C>(src, r0 - B.dist[k2], n);
      y[k2] = ld_vec<R, C>(q, r0 - B.dist[k2], n);
      b[k2] = ld_values<TV, R, NT>(val + k2 * B.ld, r0);
    }
    if constexpr (decltype(first)::value)
      if (!step()) return false;
    Vec<TV, R> sum{}, rn;
#pragma unroll
    for (int k2 = ND - 1; k2 >= 0; --k2) {
#pragma unroll
      for (int i = 0; i < R; ++i) rn.v[i] = s[k2].v[i] - al * y[k2].v[i];
      add_terms(sum, b[k2], rn);
    }
    st_vec<R, C>(dst, r0, n, rn);
    st_vec<R, C>(t, r0, n, sum);
#pragma unroll
    for (int i = 0; i < R; ++i)
      if (!C || r0 + i < n) {
        acc_prod(part[0], rn.v[i], rn.v[i]);
        acc_prod(part[1], sum.v[i], sum.v[i]);
      }
    return true;
  };
  auto any = [&](int k, auto first) -> bool {
    if (inside<R>(tl.base + tl.count - 1 - k, B.dist[ND - 1], n)) return tile(k, first, std::false_type{});
    return tile(k, first, std::true_type{});
  };
  int k = tl.first;
  const bool go = k < tl.count ? any(k, std::true_type{}) : step();
  if (go)
    for (k += tl.stride; k < tl.count; k += tl.stride) any(k, std::false_type{});
  if (l == 0 && threadIdx.x == 0) {
    State o = ld_state(&S);
    if (!was_done) {
      o.gamma = gamma;
      o.alpha = alpha;
      if (brk) {
        o.status = ST_BREAK_GAMMA;
        o.done = 1;
      }
    }
    st_state(st + 1, o);
  }
  if (!go) return;
  put_partials<2>(part, gl(v.prt), part_slot(l, grid), grid, sh);
}

// delta, beta and the stopping tests; x += alpha d; d_{i+1} = (G t + eps r) +
// beta d. G's row r reads G^T's entry (r + dist, r), which the G^T-kernel left
// in the memory-side cache. d is read and written by the row's own lane only,
// so dprev and dnext may be one buffer. Workgroup 0 publishes st[0]; the
// others read st[1] only. At 128^3 FP64 (151 MB): 24.4 -> 22.3 us.
template <typename TV, typename TG, int ND, int R, bool NT, bool HAS_EPS>
__global__ __launch_bounds__(kBlock) PCG_GT_OCCUPANCY void k_dia_G(DiaOp B, DiaVecs v, int par, int gridGT,
                                                                   int grid, uint64_t *report) {
  __shared__ Acc sh[4 * (kBlock / 64)];
  const int l = blockIdx.x, n = v.n, lane = threadIdx.x & 63;
  GLOBAL State *st = gl(v.st);
  GLOBAL const State &S = st[1];
  Acc va[2];
  load_partials<2>(gl(v.prt), gridGT, va);
  GLOBAL TV *__restrict__ x = gl((TV *)v.x);
  GLOBAL const TV *__restrict__ t = gl((const TV *)v.t);
  GLOBAL const TV *__restrict__ rc = gl((const TV *)(par ? v.r0 : v.r1));  // r_{i+1}
  GLOBAL const TV *dprev = gl((const TV *)(par ? v.d1 : v.d0));            // d_i
  GLOBAL TV *dnext = gl((TV *)(par ? v.d0 : v.d1));                        // d_{i+1}
  GLOBAL const TG *val = gl((const TG *)B.val);
  const Tiles tl = tiles_of<R>(n, l, grid);
  double delta = 0.0, eps_d = 0.0, rr = 0.0, tt = 0.0, dn = 0.0;
  TV beta = (TV)0, ap = (TV)0, eps = (TV)0;
  int status = ST_RUNNING, i1 = 0;
  bool was_done = false;
  auto step = [&]() -> bool {
    if (S.done) {  // stopped earlier, or the G^T-kernel flagged a breakdown
      was_done = true;
      return false;
    }
    delta = S.delta;
    eps_d = S.eps;
    ap = (TV)S.alpha;
    eps = (TV)eps_d;
    i1 = S.iter + 1;
    double s2[2];
    reduce_partials<2>(va, s2, sh);
    rr = s2[0];
    tt = s2[1];
    dn = tt + eps_d * rr;
    if (!(dn >= 0.0) || !isfinite(dn))
      status = ST_BREAK_DELTA;
    else if (sqrt(rr) <= S.tol_nb)
      status = ST_CONV_REC;
    else if (i1 >= S.maxit)
      status = ST_MAXIT;
    beta = (TV)(dn / delta);
    return status == ST_RUNNING;
  };
  auto tile = [&](int k, auto first, auto clamp) -> bool {
    constexpr bool C = decltype(clamp)::value;
    const int r0 = (tl.base + k) * 64 * R + lane * R;
    Vec<TV, R> b[ND], y[ND], dp, xo, r1{};
#pragma unroll
    for (int k2 = 0; k2 < ND; ++k2) {
      b[k2] = ld_values<TV, R, NT>(val + k2 * B.ld, r0 + B.dist[k2]);
      y[k2] = ld_vec<R, C>(t, r0 + B.dist[k2], n);
    }
    dp = ld_vec<R, C>(dprev, r0, n);
    xo = ld_vec<R, C>((GLOBAL const TV *)x, r0, n);
    if constexpr (HAS_EPS) r1 = ld_vec<R, C>(rc, r0, n);
    if constexpr (decltype(first)::value)
      if (!step()) return false;
    Vec<TV, R> sum{};
#pragma unroll
    for (int k2 = 0; k2 < ND; ++k2) add_terms(sum, b[k2], y[k2]);
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const TV sv = HAS_EPS ? sum.v[i] + eps * r1.v[i] : sum.v[i];
      sum.v[i] = sv + beta * dp.v[i];
      xo.v[i] = xo.v[i] + ap * dp.v[i];
    }
    st_vec<R, C>(dnext, r0, n, sum);
    st_vec<R, C>(x, r0, n, xo);
    return true;
  };
  auto any = [&](int k, auto first) -> bool {
    if (inside<R>(tl.base + k, B.dist[ND - 1], n)) return tile(k, first, std::false_type{});
    return tile(k, first, std::true_type{});
  };
  int k = tl.first;
  const bool go = k < tl.count ? any(k, std::true_type{}) : step();
  if (go)
    for (k += tl.stride; k < tl.count; k += tl.stride) any(k, std::false_type{});
  if (l == 0 && threadIdx.x == 0) {
    State o = ld_state(&S);
    if (!was_done) {
      o.rr = rr;
      o.tt = tt;
      o.iter = i1;
      o.alpha = 0.0;  // x += alpha_i d_i is applied in this kernel, whatever the status
      if (status != ST_BREAK_DELTA) {
        o.beta = dn / delta;
        o.delta = dn;
      }
      if (status != ST_RUNNING) {
        o.status = status;
        o.done = 1;
      }
    }
    st_state(st, o);
    report_progress(report, o.iter, o.done);
  }
  if (!go && !was_done) {  // stopped: x_{i+1} only
    int64_t i0, i1r;
    ew_rows(n, l, grid, i0, i1r);
    for (int64_t i = i0 + threadIdx.x; i < i1r; i += kBlock) x[i] = x[i] + ap * dprev[i];
  }
}

// Stencil storage from a matrix placed in sliced diagonals (M.val raw, TU the
// unsigned type of its width): entry (r, r - dist[k]) to val[k ld + r], zero
// where there is none and for the rows beyond n.
template <typename TU>
__global__ __launch_bounds__(kBlock) void k_dia_build(DevCSR M, DiaOp o) {
  GLOBAL const int32_t *blk = gl(M.blk), *off = gl(M.ci);
  GLOBAL const TU *src = gl((const TU *)M.val);
  GLOBAL TU *dst = gl((TU *)o.val);
  for (int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x; r < o.ld; r += (int64_t)gridDim.x * kBlock) {
    int a = 0, e = 0;
    if (r < M.n) {
      a = blk[r / kSliceRows];
      e = blk[r / kSliceRows + 1];
    }
    for (int k = 0; k < o.nd; ++k) {
      TU u = 0;
      for (int p = a; p < e; ++p)
        if (off[p] == -o.dist[k]) u = src[(int64_t)p * kSliceRows + r % kSliceRows];
      dst[k * o.ld + r] = u;
    }
  }
}

// flag[0] = 1 unless M's entries (r, r + dist[k]) equal the stored (r + dist[k], r)
// bit for bit for every row r and every diagonal k > 0 (an absent entry is a zero).
template <typename TU>
__global__ __launch_bounds__(kBlock) void k_dia_symmetric(DevCSR M, DiaOp o, int32_t *flag_) {
  GLOBAL const int32_t *blk = gl(M.blk), *off = gl(M.ci);
  GLOBAL const TU *src = gl((const TU *)M.val);
  GLOBAL const TU *low = gl((const TU *)o.val);
  for (int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x; r < M.n; r += (int64_t)gridDim.x * kBlock) {
    const int a = blk[r / kSliceRows], e = blk[r / kSliceRows + 1];
    for (int k = 1; k < o.nd; ++k) {
      TU u = 0;
      for (int p = a; p < e; ++p)
        if (off[p] == o.dist[k]) u = src[(int64_t)p * kSliceRows + r % kSliceRows];
      if (u != low[k * o.ld + r + o.dist[k]]) gl(flag_)[0] = 1;
    }
  }
}

// ---------------------------------------------------------------- launchers

#define PCG_DIA_LAUNCH(kern, grid, ...)                                                         \
  do {                                                                                          \
    if (e0 || e1)                                                                               \
      hipExtLaunchKernelGGL(kern, dim3(grid), dim3(kBlock), 0, s, e0, e1, 0, __VA_ARGS__);      \
    else                                                                                        \
      hipLaunchKernelGGL(kern, dim3(grid), dim3(kBlock), 0, s, __VA_ARGS__);                    \
  } while (0)

#define PCG_DIA_ND(nd_, ND, ...)                           \
  switch (nd_) {                                           \
    case 1: { constexpr int ND = 1; __VA_ARGS__; break; }  \
    case 2: { constexpr int ND = 2; __VA_ARGS__; break; }  \
    case 3: { constexpr int ND = 3; __VA_ARGS__; break; }  \
    case 4: { constexpr int ND = 4; __VA_ARGS__; break; }  \
    case 5: { constexpr int ND = 5; __VA_ARGS__; break; }  \
    default: return hipErrorInvalidValue;                  \
  }

// G's storage types (with FP32 vectors G is not FP64).
#define PCG_DIA_G(gdt, TG, ...)                                \
  switch (gdt) {                                               \
    case F64: { using TG = double; __VA_ARGS__; break; }       \
    case F32: { using TG = float; __VA_ARGS__; break; }        \
    case BF16: { using TG = bf16_t; __VA_ARGS__; break; }      \
    case F16: { using TG = _Float16; __VA_ARGS__; break; }     \
    default: return hipErrorInvalidValue;                      \
  }

hipError_t launch_dia_A(const Types &ty, const DiaOp &A, const DiaVecs &v, int par, int grid, hipStream_t s,
                        hipEvent_t e0, hipEvent_t e1) {
  if (ty.vec != ty.a) return hipErrorInvalidValue;
  PCG_DIA_ND(A.nd, ND, {
    if (ty.vec == F64) {
      if (A.temporal)
        PCG_DIA_LAUNCH((k_dia_A<double, double, ND, kDiaR64, false>), grid, A, v, par, grid);
      else
        PCG_DIA_LAUNCH((k_dia_A<double, double, ND, kDiaR64, true>), grid, A, v, par, grid);
    } else {
      if (A.temporal)
        PCG_DIA_LAUNCH((k_dia_A<float, float, ND, kDiaR32, false>), grid, A, v, par, grid);
      else
        PCG_DIA_LAUNCH((k_dia_A<float, float, ND, kDiaR32, true>), grid, A, v, par, grid);
    }
  });
  return hipGetLastError();
}

hipError_t launch_dia_GT(const Types &ty, const DiaOp &B, const DiaVecs &v, int par, int gridA, int grid,
                         hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  if (ty.vec == F32 && ty.g == F64) return hipErrorInvalidValue;
  PCG_DIA_ND(B.nd, ND, PCG_DIA_G(ty.g, TG, {
    if (ty.vec == F64) {
      if (B.temporal)
        PCG_DIA_LAUNCH((k_dia_GT<double, TG, ND, kDiaR64, false>), grid, B, v, par, gridA, grid);
      else
        PCG_DIA_LAUNCH((k_dia_GT<double, TG, ND, kDiaR64, true>), grid, B, v, par, gridA, grid);
    } else if constexpr (!std::is_same_v<TG, double>) {
      if (B.temporal)
        PCG_DIA_LAUNCH((k_dia_GT<float, TG, ND, kDiaR32, false>), grid, B, v, par, gridA, grid);
      else
        PCG_DIA_LAUNCH((k_dia_GT<float, TG, ND, kDiaR32, true>), grid, B, v, par, gridA, grid);
    }
  }));
  return hipGetLastError();
}

template <typename TV, typename TG, int ND, int R>
static hipError_t launch_g(const DiaOp &B, const DiaVecs &v, bool has_eps, int par, int gridGT, int grid,
                           hipStream_t s, hipEvent_t e0, hipEvent_t e1, uint64_t *report) {
  if (has_eps) {
    if (B.temporal)
      PCG_DIA_LAUNCH((k_dia_G<TV, TG, ND, R, false, true>), grid, B, v, par, gridGT, grid, report);
    else
      PCG_DIA_LAUNCH((k_dia_G<TV, TG, ND, R, true, true>), grid, B, v, par, gridGT, grid, report);
  } else {
    if (B.temporal)
      PCG_DIA_LAUNCH((k_dia_G<TV, TG, ND, R, false, false>), grid, B, v, par, gridGT, grid, report);
    else
      PCG_DIA_LAUNCH((k_dia_G<TV, TG, ND, R, true, false>), grid, B, v, par, gridGT, grid, report);
  }
  return hipGetLastError();
}

hipError_t launch_dia_G(const Types &ty, const DiaOp &B, const DiaVecs &v, bool has_eps, int par, int gridGT, int grid,
                        hipStream_t s, hipEvent_t e0, hipEvent_t e1, uint64_t *report) {
  PCG_DIA_ND(B.nd, ND, PCG_DIA_G(ty.g, TG, {
    if (ty.vec == F64) return launch_g<double, TG, ND, kDiaR64>(B, v, has_eps, par, gridGT, grid, s, e0, e1, report);
    if constexpr (!std::is_same_v<TG, double>)
      return launch_g<float, TG, ND, kDiaR32>(B, v, has_eps, par, gridGT, grid, s, e0, e1, report);
  }));
  return hipErrorInvalidValue;
}

hipError_t launch_dia_build(const DevCSR &M, const DiaOp &o, int32_t *flag, hipStream_t s) {
  const int grid = (int)std::min<int64_t>((o.ld + kBlock - 1) / kBlock, 8192);
  switch (dtype_size(M.dtype)) {
    case 8: hipLaunchKernelGGL((k_dia_build<uint64_t>), dim3(grid), dim3(kBlock), 0, s, M, o); break;
    case 4: hipLaunchKernelGGL((k_dia_build<uint32_t>), dim3(grid), dim3(kBlock), 0, s, M, o); break;
    default: hipLaunchKernelGGL((k_dia_build<uint16_t>), dim3(grid), dim3(kBlock), 0, s, M, o); break;
  }
  if (flag) {
    if (dtype_size(M.dtype) == 8)
      hipLaunchKernelGGL((k_dia_symmetric<uint64_t>), dim3(grid), dim3(kBlock), 0, s, M, o, flag);
    else if (dtype_size(M.dtype) == 4)
      hipLaunchKernelGGL((k_dia_symmetric<uint32_t>), dim3(grid), dim3(kBlock), 0, s, M, o, flag);
    else
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace pcgk
