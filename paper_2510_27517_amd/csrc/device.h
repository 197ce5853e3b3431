// Device-side building blocks shared by the gfx950 kernels: matrix access in
// every storage layout (rows summed left to right in CSR order), inner
// products in double-double sums, and the placement of a system's work on workgroups. The layouts
// are described at DevCSR.
#pragma once
#include <hip/hip_runtime.h>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "kernels.h"

namespace pcgk {

// The SpMV kernels are memory-latency bound: they are compiled for 8 waves
// per SIMD (at most 64 VGPRs, checked free of scratch spills), which keeps
// twice the loads in flight of the 4-6 waves the compiler otherwise picks.
#ifndef PCG_WAVES_PER_EU
#define PCG_WAVES_PER_EU 8
#endif
#define PCG_OCCUPANCY __attribute__((amdgpu_waves_per_eu(PCG_WAVES_PER_EU)))
// The G^T-kernel takes two rows per lane over sliced diagonals (twice the
// operands per lane): compiled for 4 waves per SIMD (at most 128 VGPRs, no
// spills), the occupancy its default grid of 4 workgroups of 4 waves per CU
// gives anyway.
#define PCG_GT_OCCUPANCY __attribute__((amdgpu_waves_per_eu(4)))
// The G-kernel takes two rows per lane over sliced diagonals too and holds
// its first slice pair's operands while its workgroup reduces the partial
// sums of the G^T-kernel: compiled for 4 waves per SIMD like the G^T-kernel.
#define PCG_G_OCCUPANCY __attribute__((amdgpu_waves_per_eu(4)))

struct bf16_t { uint16_t bits; };

// Pointers that come out of the device directory are not known to the
// compiler to address global memory, and accesses through them compile to
// flat instructions, which also count on the LDS wait counter and so stall
// every LDS wait of the staging loop behind outstanding gathers. Kernels
// therefore take every directory pointer into the global address space.
#define GLOBAL __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ GLOBAL T *gl(T *p) {
  return (GLOBAL T *)p;
}

// Layout metadata that a whole wave reads at one address (slice pointers,
// per-slice column offsets) is read through the constant address space, so
// that those reads compile to scalar loads: they wait on their own counter
// instead of behind the wave's outstanding vector loads and stores. Valid
// because no kernel writes a layout's metadata while it is being read.
#define CONSTANT __attribute__((address_space(4)))
template <typename T>
__device__ __forceinline__ CONSTANT const T *ro(GLOBAL const T *p) {
  return (CONSTANT const T *)p;
}

// Matrix values and column indices are read once per product. NT = true:
// nontemporal loads, which stream past the caches (they neither displace the
// gathered vector entries in L2 nor stay in the memory-side cache); NT =
// false: ordinary loads, for a matrix meant to stay resident in the 256 MB
// memory-side cache from one iteration to the next (DevCSR::temporal).
template <bool NT = true, typename T>
__device__ __forceinline__ T ldstream(GLOBAL const T *p, int64_t k) {
  if constexpr (NT)
    return __builtin_nontemporal_load(p + k);
  else
    return p[k];
}

template <bool NT = true>
__device__ __forceinline__ double ldval(GLOBAL const double *p, int64_t k) {
  return ldstream<NT>(p, k);
}
template <bool NT = true>
__device__ __forceinline__ float ldval(GLOBAL const float *p, int64_t k) {
  return ldstream<NT>(p, k);
}
template <bool NT = true>
__device__ __forceinline__ float ldval(GLOBAL const bf16_t *p, int64_t k) {
  return __uint_as_float((uint32_t)ldstream<NT>((GLOBAL const uint16_t *)p, k) << 16);
}
template <bool NT = true>
__device__ __forceinline__ float ldval(GLOBAL const _Float16 *p, int64_t k) {
  return (float)ldstream<NT>(p, k);
}

// Whole-record copies of a State (one thread publishes a slot), in 16-byte
// words of a builtin vector type (usable in any address space).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ State ld_state(GLOBAL const State *p) {
  constexpr int W = (int)(sizeof(State) / 16);
  u32x4 w[W];
  GLOBAL const u32x4 *q = (GLOBAL const u32x4 *)p;
#pragma unroll
  for (int i = 0; i < W; ++i) w[i] = q[i];
  State o;
  __builtin_memcpy(&o, w, sizeof(State));
  return o;
}

__device__ __forceinline__ void st_state(GLOBAL State *p, const State &o) {
  constexpr int W = (int)(sizeof(State) / 16);
  u32x4 w[W];
  __builtin_memcpy(w, &o, sizeof(State));
  GLOBAL u32x4 *q = (GLOBAL u32x4 *)p;
#pragma unroll
  for (int i = 0; i < W; ++i) q[i] = w[i];
}

template <typename TM>
struct Mat {
  GLOBAL const int32_t *rp;
  GLOBAL const int32_t *ci;
  GLOBAL const TM *val;
  GLOBAL const int32_t *blk;
  int32_t nblk;
  int32_t n;
  int32_t fmt;
  int32_t idx16;
  int32_t temporal;
  int32_t rpl;
};

// FMT >= 0: a kernel built for that layout alone, which leaves the others' code
// and registers out of it.
template <typename TM, int FMT = -1>
__device__ __forceinline__ Mat<TM> mat(const DevCSR &m) {
  return Mat<TM>{gl(m.rp),   gl(m.ci), gl((const TM *)m.val), gl(m.blk), m.nblk, m.n, FMT >= 0 ? FMT : m.fmt,
                 m.idx16, m.temporal, m.rpl};
}

// Column of stored entry q of `row`: an absolute int32 index, or (sliced
// layouts with 16-bit indices) an int16 difference from the row.
template <typename TI>
__device__ __forceinline__ int32_t col_at(GLOBAL const int32_t *ci, int64_t q, int32_t row) {
  if constexpr (sizeof(TI) == 2)
    return row + (int32_t)((GLOBAL const int16_t *)ci)[q];
  else
    return ci[q];
}

// Operands of one row loaded before the row's products are staged.
template <typename TV>
struct RowVals {
  TV a, b, c;
};

// Sum of lds[a..e) added left to right onto s0; eight reads are issued ahead
// of their adds, so long rows are not one LDS round trip per entry.
template <typename TACC>
__device__ __forceinline__ TACC lds_row_sum(const TACC *lds, int a, int e, TACC s0 = 0) {
  TACC sum = s0;
  int k = a;
  for (; k + 8 <= e; k += 8) {
    TACC v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = lds[k + u];
#pragma unroll
    for (int u = 0; u < 8; ++u) sum += v[u];
  }
  for (; k < e; ++k) sum += lds[k];
  return sum;
}

// Products [c0, c1) of a row block into LDS (from c0's slot on). What bounds a
// block is two dependent memory latencies per round (column, then gather).
// U > 1: each thread takes U entries a round with all their loads in flight; a
// round's surplus repeats the last entry (in bounds) and is not stored. U = 0, 1:
// a plain loop unrolled by four, whose remainder runs one entry after the other
// (1: with the block's bounds from scalar loads, as for U > 1).
// Which is faster depends on the kernel's types: see the kernels' US.
template <typename TACC, int U, bool NT, typename TM, typename Gather>
__device__ __forceinline__ void stage_products(const Mat<TM> &M, int c0, int c1, TACC *lds, Gather gather) {
  // entries count from the block's first: nonzeros number up to 2^31 - 1, and a
  // round's step past the last of them must not wrap below zero (counted from the
  // matrix's first in unsigned, 72,000 rows of 470 took 582 us per iteration in
  // FP64 and 434 in FP32 against 561 and 414)
  const int m = c1 - c0;
  if constexpr (U <= 1) {
#pragma unroll 4
    for (int k = (int)threadIdx.x; k < m; k += kBlock)
      lds[k] = (TACC)ldval<NT>(M.val, (int64_t)c0 + k) * gather(ldstream<NT>(M.ci, (int64_t)c0 + k));
  } else {
    for (int c = (int)threadIdx.x; c < m; c += U * kBlock) {
      int32_t col[U];
      TACC v[U];
      decltype(gather(0)) x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t k = (int64_t)c0 + min(c + u * kBlock, m - 1);
        col[u] = ldstream<NT>(M.ci, k);
        v[u] = (TACC)ldval<NT>(M.val, k);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) x[u] = gather(col[u]);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (c + u * kBlock < m) lds[c + u * kBlock] = v[u] * x[u];
    }
  }
}

// One row block: stage products in LDS, sum each row in CSR order. `pre(row)`
// loads the row's own operands early (overlapping the gathers), `epi(row,
// sum, pre_values)` consumes the row's sum. hook: a workgroup step between
// the products and the first epilogue (it may hold barriers); false ends the
// walk.
template <typename TACC, int U, bool NT, typename TM, typename Pre, typename Gather, typename Epi, typename Hook>
__device__ __forceinline__ bool stream_block(const Mat<TM> &M, int b, TACC *lds, Pre pre, Gather gather, Epi epi,
                                             Hook hook) {
  constexpr int cap = kLdsBytes / (int)sizeof(TACC);
  const int tid = threadIdx.x;
  int r0, k0, r1, k1;
  if constexpr (U == 0) {
    r0 = M.blk[2 * b], k0 = M.blk[2 * b + 1], r1 = M.blk[2 * b + 2], k1 = M.blk[2 * b + 3];
  } else {  // scalar loads
    CONSTANT const int32_t *blk = ro(M.blk) + 2 * b;
    r0 = blk[0], k0 = blk[1], r1 = blk[2], k1 = blk[3];
  }
  if (k1 - k0 <= cap) {
    const int row = r0 + tid;
    const bool has = row < r1;
    int a = 0, e = 0;
    RowVals<TACC> pv{};
    if (has) {
      a = M.rp[row] - k0;
      e = M.rp[row + 1] - k0;
      pv = pre(row);
    }
    stage_products<TACC, U, NT>(M, k0, k1, lds, gather);
    if (!hook()) return false;
    __syncthreads();
    if (has) epi(row, lds_row_sum(lds, a, e), pv);
    __syncthreads();
  } else {
    // a single row longer than the LDS window: chunks, summed in order by thread 0
    RowVals<TACC> pv{};
    if (tid == 0) pv = pre(r0);
    TACC sum = 0;
    for (int c0 = k0; c0 < k1; c0 += cap) {
      const int c1 = min(c0 + cap, k1);
      stage_products<TACC, U, NT>(M, c0, c1, lds, gather);
      __syncthreads();
      if (tid == 0) sum = lds_row_sum(lds, 0, c1 - c0, sum);
      __syncthreads();
    }
    if (!hook()) return false;
    if (tid == 0) epi(r0, sum, pv);
  }
  return true;
}

struct NoHook {
  __device__ __forceinline__ bool operator()() const { return true; }
};

// This workgroup's row blocks: first, first + stride, ... < end; L is its
// logical index (the slot of its partial sums). l is the workgroup's index
// among its system's G workgroups (G and the system's first workgroup are
// multiples of 8, so l % 8 is the XCD the workgroup runs on).
struct Sched {
  int first, end, stride, L;
};

__device__ __forceinline__ Sched sched(int nblk, int l, int G) {
  const int W = G >> 3, x = l & 7, w = l >> 3;
  Sched sc;
  sc.first = (int)((int64_t)x * nblk / 8) + w;
  sc.end = (int)((int64_t)(x + 1) * nblk / 8);
  sc.stride = W;
  sc.L = x * W + w;
  return sc;
}

// Slot of this workgroup's partial sums (the same for both layouts).
__device__ __forceinline__ int part_slot(int l, int G) { return (l & 7) * (G >> 3) + (l >> 3); }

// Column of a slice entry: an absolute int32 index, or an int16 difference
// from the lane's row.
template <bool NT>
__device__ __forceinline__ int32_t slice_col(GLOBAL const int32_t *cc, int64_t k, int32_t) {
  return ldstream<NT>(cc, k);
}
template <bool NT>
__device__ __forceinline__ int32_t slice_col(GLOBAL const int16_t *cc, int64_t k, int32_t row) {
  return row + (int32_t)ldstream<NT>(cc, k);
}

// One lane's row of a slice: products of its wd entries added left to right
// from zero, loads issued UNR at a time. The last wd % UNR entries form one
// more batch whose surplus loads repeat entry wd - 1 (in bounds) and whose
// surplus products are not added, so every load of a batch is in flight at
// once (wd is the same for the whole wave).
template <typename TACC, int UNR, bool NT, typename TM, typename TI, typename Gather>
__device__ __forceinline__ TACC slice_row_sum(GLOBAL const TM *vv, GLOBAL const TI *cc, int32_t row, int wd,
                                              Gather gather) {
  TACC sum = 0;
  int k = 0;
  for (; k + UNR <= wd; k += UNR) {
    TACC p[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u)
      p[u] = (TACC)ldval<NT>(vv, (k + u) * kSliceRows) * gather(slice_col<NT>(cc, (k + u) * kSliceRows, row));
#pragma unroll
    for (int u = 0; u < UNR; ++u) sum += p[u];
  }
  const int rem = wd - k;
  if (rem > 0) {
    TACC p[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int e = k + min(u, rem - 1);
      p[u] = (TACC)ldval<NT>(vv, e * kSliceRows) * gather(slice_col<NT>(cc, e * kSliceRows, row));
    }
#pragma unroll
    for (int u = 0; u < UNR; ++u)
      if (u < rem) sum += p[u];
  }
  return sum;
}

template <typename TACC, int UW, bool NT, typename TM, typename TI, typename Gather>
__device__ __forceinline__ TACC slice_row(GLOBAL const TM *vv, GLOBAL const TI *cc, int32_t row, int wd,
                                          Gather gather) {
  return (UW > 4 && wd > 4) ? slice_row_sum<TACC, UW, NT>(vv, cc, row, wd, gather)
                            : slice_row_sum<TACC, 4, NT>(vv, cc, row, wd, gather);
}

// Sliced-ELL rows: each wave takes whole slices (64 rows, one per lane); a
// lane loads its row's entries with coalesced loads across the slice, gathers,
// and adds the products left to right from zero, the CSR order. No LDS and no
// barrier. The XCD slab split is the one of the row blocks.
// UW: loads in flight per lane for rows longer than 4 entries (8 pays where a
// row product gathers one vector and the epilogue holds few operands; under
// the 64-register budget kernels with two gathers per entry do better with 4).
// REV: each die walks its range of slices from the top down.
template <typename TACC, int UW, bool NT, bool REV, typename TM, typename Pre, typename Gather, typename Epi>
__device__ __forceinline__ void sell_rows(const Mat<TM> &M, int l, int G, Pre pre, Gather gather, Epi epi) {
  constexpr int NW = kBlock / 64;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int W = G >> 3, x = l & 7, w = l >> 3;
  const int s0 = (int)((int64_t)x * M.nblk / 8), s1 = (int)((int64_t)(x + 1) * M.nblk / 8);
  for (int k = w * NW + wv; k < s1 - s0; k += W * NW) {
    const int c = REV ? s1 - 1 - k : s0 + k;
    const int o0 = ro(M.blk)[c], wd = ro(M.blk)[c + 1] - o0;
    const int row = c * kSliceRows + lane;
    const bool has = row < M.n;
    RowVals<TACC> pv{};
    if (has) pv = pre(row);
    const int64_t o = (int64_t)o0 * kSliceRows + lane;
    GLOBAL const TM *vv = M.val + o;
    const TACC sum = M.idx16 ? slice_row<TACC, UW, NT>(vv, (GLOBAL const int16_t *)M.ci + o, row, wd, gather)
                             : slice_row<TACC, UW, NT>(vv, M.ci + o, row, wd, gather);
    if (has) epi(row, sum, pv);
  }
}

// sell_rows with a workgroup step (hook) between the first slice's products and
// its epilogue, as in sdia_rows_h.
template <typename TACC, int UW, bool NT, bool REV, typename TM, typename Pre, typename Gather, typename Epi,
          typename Hook>
__device__ __forceinline__ bool sell_rows_h(const Mat<TM> &M, int l, int G, Pre pre, Gather gather, Epi epi, Hook hook) {
  constexpr int NW = kBlock / 64;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int W = G >> 3, x = l & 7, w = l >> 3;
  const int s0 = (int)((int64_t)x * M.nblk / 8), s1 = (int)((int64_t)(x + 1) * M.nblk / 8);
  auto slice = [&](int k, auto first) -> bool {
    const int c = REV ? s1 - 1 - k : s0 + k;
    const int o0 = ro(M.blk)[c], wd = ro(M.blk)[c + 1] - o0;
    const int row = c * kSliceRows + lane;
    const bool has = row < M.n;
    RowVals<TACC> pv{};
    if (has) pv = pre(row);
    const int64_t o = (int64_t)o0 * kSliceRows + lane;
    GLOBAL const TM *vv = M.val + o;
    const TACC sum = M.idx16 ? slice_row<TACC, UW, NT>(vv, (GLOBAL const int16_t *)M.ci + o, row, wd, gather)
                             : slice_row<TACC, UW, NT>(vv, M.ci + o, row, wd, gather);
    if constexpr (decltype(first)::value)
      if (!hook()) return false;
    if (has) epi(row, sum, pv);
    return true;
  };
  int k = w * NW + wv;
  if (k >= s1 - s0) return hook();
  if (!slice(k, std::true_type{})) return false;
  for (k += W * NW; k < s1 - s0; k += W * NW) slice(k, std::false_type{});
  return true;
}

// One lane's row of a sliced-diagonal slice: value k of the row multiplies
// the gathered entry at column row + off[k] (clamped into [0, n): a stored
// zero's column may fall outside), added left to right from zero; loads
// issued UNR at a time as in slice_row_sum. off[] is the same for the whole
// wave (scalar loads).
template <typename TACC, int UNR, bool NT, bool DIAG = false, typename TM, typename Gather>
__device__ __forceinline__ TACC sdia_row_sum(GLOBAL const TM *vv, CONSTANT const int32_t *off, int32_t row, int32_t nmax,
                                             int wd, Gather gather, TACC dg = 0) {
  // DIAG: dg is the operand at the row's own column (offset 0), already
  // loaded by the caller, so that entry is not gathered again
  auto operand = [&](int32_t o) -> TACC {
    if constexpr (DIAG) {
      if (o == 0) return dg;
    }
    return gather(min(max(row + o, 0), nmax));
  };
  TACC sum = 0;
  int k = 0;
  for (; k + UNR <= wd; k += UNR) {
    TACC p[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) p[u] = (TACC)ldval<NT>(vv, (k + u) * kSliceRows) * operand(off[k + u]);
#pragma unroll
    for (int u = 0; u < UNR; ++u) sum += p[u];
  }
  const int rem = wd - k;
  if (rem > 0) {
    TACC p[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int e = k + min(u, rem - 1);
      p[u] = (TACC)ldval<NT>(vv, e * kSliceRows) * operand(off[e]);
    }
#pragma unroll
    for (int u = 0; u < UNR; ++u)
      if (u < rem) sum += p[u];
  }
  return sum;
}

// Sliced-diagonal rows: the walk of sell_rows (whole slices per wave, one
// lane per row, each die's eighth of the slices), with one column offset per
// slice entry instead of one index per lane.
template <typename TACC, int UW, bool NT, bool REV, bool DIAG = false, typename TM, typename Pre, typename Gather,
          typename Epi>
__device__ __forceinline__ void sdia_rows(const Mat<TM> &M, int l, int G, Pre pre, Gather gather, Epi epi) {
  constexpr int NW = kBlock / 64;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int W = G >> 3, x = l & 7, w = l >> 3;
  const int s0 = (int)((int64_t)x * M.nblk / 8), s1 = (int)((int64_t)(x + 1) * M.nblk / 8);
  for (int k = w * NW + wv; k < s1 - s0; k += W * NW) {
    const int c = REV ? s1 - 1 - k : s0 + k;
    const int o0 = ro(M.blk)[c], wd = ro(M.blk)[c + 1] - o0;
    const int row = c * kSliceRows + lane;
    const bool has = row < M.n;
    RowVals<TACC> pv{};
    if (has) pv = pre(row);
    GLOBAL const TM *vv = M.val + (int64_t)o0 * kSliceRows + lane;
    const TACC sum = (UW > 4 && wd > 4)
                         ? sdia_row_sum<TACC, UW, NT, DIAG>(vv, ro(M.ci) + o0, row, M.n - 1, wd, gather, pv.a)
                         : sdia_row_sum<TACC, 4, NT, DIAG>(vv, ro(M.ci) + o0, row, M.n - 1, wd, gather, pv.a);
    if (has) epi(row, sum, pv);
  }
}

// sdia_rows with a workgroup step between the first slice's products and its
// epilogue: every wave calls hook() exactly once (after the loop when it has
// no slice), so hook may hold barriers; its result, the same in every thread,
// says whether the walk goes on. A kernel that needs a reduction before its
// epilogue (the G-kernel's beta) issues its first slice's loads and products
// under that reduction's latency instead of after it.
template <typename TACC, int UW, bool NT, bool REV, typename TM, typename Pre, typename Gather, typename Epi,
          typename Hook>
__device__ __forceinline__ bool sdia_rows_h(const Mat<TM> &M, int l, int G, Pre pre, Gather gather, Epi epi,
                                            Hook hook) {
  constexpr int NW = kBlock / 64;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int W = G >> 3, x = l & 7, w = l >> 3;
  const int s0 = (int)((int64_t)x * M.nblk / 8), s1 = (int)((int64_t)(x + 1) * M.nblk / 8);
  // the first slice is peeled so that what hook needs is dead in the loop
  auto slice = [&](int k, auto first) -> bool {
    const int c = REV ? s1 - 1 - k : s0 + k;
    const int o0 = ro(M.blk)[c], wd = ro(M.blk)[c + 1] - o0;
    const int row = c * kSliceRows + lane;
    const bool has = row < M.n;
    RowVals<TACC> pv{};
    if (has) pv = pre(row);
    GLOBAL const TM *vv = M.val + (int64_t)o0 * kSliceRows + lane;
    const TACC sum = (UW > 4 && wd > 4) ? sdia_row_sum<TACC, UW, NT>(vv, ro(M.ci) + o0, row, M.n - 1, wd, gather)
                                        : sdia_row_sum<TACC, 4, NT>(vv, ro(M.ci) + o0, row, M.n - 1, wd, gather);
    if constexpr (decltype(first)::value)
      if (!hook()) return false;
    if (has) epi(row, sum, pv);
    return true;
  };
  int k = w * NW + wv;
  if (k >= s1 - s0) return hook();
  if (!slice(k, std::true_type{})) return false;
  for (k += W * NW; k < s1 - s0; k += W * NW) slice(k, std::false_type{});
  return true;
}

// ---- two rows per lane over sliced diagonals
//
// Rows r and r + 1 of a slice read their operands at one offset o from the
// adjacent entries r + o and r + 1 + o, their values from adjacent slots,
// and write adjacent results: a lane that owns both rows makes one access of
// twice the width for each, half the memory instructions of one row per
// lane (gathers, the bulk of them, are unaligned 8- or 16-byte loads).

// Two adjacent entries of a vector (any alignment of the element type).
template <typename T>
struct Pair {
  T x, y;
};
template <typename T>
__device__ __forceinline__ Pair<T> ld_pair(GLOBAL const T *p, int64_t i) {
  Pair<T> v;
  __builtin_memcpy(&v, p + i, sizeof(v));
  return v;
}
template <typename T>
__device__ __forceinline__ void st_pair(GLOBAL T *p, int64_t i, T a, T b) {
  const Pair<T> v{a, b};
  __builtin_memcpy(p + i, &v, sizeof(v));
}

// The operands of rows r0 and r0 + 1 at column offset o, j0 = r0 + o: the
// entries at j0 and j0 + 1, each clamped into [0, n) as the one-row walk
// clamps it, from one load of [lo, lo + 1] (n >= 2).
template <typename T>
__device__ __forceinline__ Pair<T> gather_pair(GLOBAL const T *x, int32_t j0, int32_t n) {
  const int32_t lo = min(max(j0, 0), n - 2);
  const Pair<T> v = ld_pair(x, lo);
  return Pair<T>{j0 > n - 2 ? v.y : v.x, j0 < 0 ? v.x : v.y};
}

// Values of two adjacent slots (an even slot of a 64-slot slice entry:
// aligned to twice the value size), with the matrix's load policy.
typedef double v2f64 __attribute__((ext_vector_type(2)));
typedef float v2f32 __attribute__((ext_vector_type(2)));
typedef _Float16 v2f16 __attribute__((ext_vector_type(2)));
template <bool NT, typename V>
__device__ __forceinline__ V ld_aligned(GLOBAL const V *p) {
  if constexpr (NT)
    return __builtin_nontemporal_load(p);
  else
    return *p;
}
template <bool NT, typename TACC>
__device__ __forceinline__ void ldval_pair(GLOBAL const double *p, int64_t k, TACC &a, TACC &b) {
  const v2f64 v = ld_aligned<NT>((GLOBAL const v2f64 *)(p + k));
  a = (TACC)v.x;
  b = (TACC)v.y;
}
template <bool NT, typename TACC>
__device__ __forceinline__ void ldval_pair(GLOBAL const float *p, int64_t k, TACC &a, TACC &b) {
  const v2f32 v = ld_aligned<NT>((GLOBAL const v2f32 *)(p + k));
  a = (TACC)v.x;
  b = (TACC)v.y;
}
template <bool NT, typename TACC>
__device__ __forceinline__ void ldval_pair(GLOBAL const bf16_t *p, int64_t k, TACC &a, TACC &b) {
  const uint32_t v = ld_aligned<NT>((GLOBAL const uint32_t *)(p + k));
  a = (TACC)__uint_as_float(v << 16);
  b = (TACC)__uint_as_float(v & 0xffff0000u);
}
template <bool NT, typename TACC>
__device__ __forceinline__ void ldval_pair(GLOBAL const _Float16 *p, int64_t k, TACC &a, TACC &b) {
  const v2f16 v = ld_aligned<NT>((GLOBAL const v2f16 *)(p + k));
  a = (TACC)(float)v.x;
  b = (TACC)(float)v.y;
}

// Sliced-diagonal rows, two per lane: a wave takes two slices at once (lanes
// 0-31 the first, 32-63 the second; in each die's range, pairs of slices
// from the bottom up, or the top down with REV), lane L rows 2 (L mod 32)
// and 2 (L mod 32) + 1 of its slice. Each row's products are added left to
// right from zero, as in the one-row walk, so both walks give the same bits.
// The kernel's functors work on row pairs:
//   pre2(r0, h0, h1) -> the pair's own operands (rows r0, r0 + 1; h0, h1:
//                       whether each row exists),
//   load2(j0)        -> what the operands at columns j0, j0 + 1 are made of
//                       (clamped loads, gather_pair),
//   comb2(loaded)    -> Pair<TACC>, those operands,
//   epi2(r0, h0, h1, sum0, sum1, pre_values),
// PRE_AT_DIAG: pre2 returns what load2(r0) would, on every row the epilogue
// keeps, so a leading entry at offset 0 (a diagonal) reuses it instead of
// loading the same operands again.
//   hook()           -> a workgroup step, called by every wave exactly once:
//                       after its first slice pair's loads are issued and
//                       before anything uses them (after the loop when the
//                       wave has no slice), so it may hold barriers and
//                       compute what comb2 needs; its result, the same in
//                       every thread, says whether the walk goes on.
// n >= 2.
template <typename TACC, bool NT, bool REV, bool PRE_AT_DIAG, typename TM, typename Pre2, typename Load2,
          typename Comb2, typename Epi2, typename Hook>
__device__ __forceinline__ bool sdia_rows2(const Mat<TM> &M, int l, int G, Pre2 pre2, Load2 load2, Comb2 comb2,
                                           Epi2 epi2, Hook hook) {
  constexpr int NW = kBlock / 64, U = 4;
  const int lane = threadIdx.x & 63, half = lane >> 5, lr = 2 * (lane & 31);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int W = G >> 3, x = l & 7, w = l >> 3;
  const int s0 = (int)((int64_t)x * M.nblk / 8), s1 = (int)((int64_t)(x + 1) * M.nblk / 8);
  const int npairs = (s1 - s0 + 1) / 2;
  // the first pair and its first chunk of entries are peeled so that what
  // hook needs is dead in the loops
  auto pair = [&](int p, auto first) -> bool {
    // slices ca (lanes 0-31) and cb = ca + 1 (lanes 32-63); at an odd end of
    // the range one of them lies outside it and its lanes idle on the other
    const int ca = REV ? s1 - 2 - 2 * p : s0 + 2 * p, cb = ca + 1;
    const bool va = ca >= s0, vb = cb < s1;
    // both slices' pointers and offsets are read whole-wave (scalar loads);
    // each half selects its own slice (cb <= s1 <= nblk, so blk[cb] exists)
    CONSTANT const int32_t *blk = ro(M.blk), *ci = ro(M.ci);
    const int ob = blk[cb], oa = va ? blk[ca] : ob, oe = vb ? blk[cb + 1] : ob;
    const int wa = ob - oa, wb = oe - ob;
    const bool useb = half ? vb : !va;
    const bool live = half ? vb : va;
    const int cs = useb ? cb : ca, o0 = useb ? ob : oa, wd = useb ? wb : wa;
    const int wmax = max(wa, wb);
    const int r0 = cs * kSliceRows + lr;
    const bool h0 = live && r0 < M.n, h1 = live && r0 + 1 < M.n;
    const auto pv = pre2(r0, h0, h1);
    GLOBAL const TM *vv = M.val + (int64_t)o0 * kSliceRows + lr;
    TACC sa = 0, sb = 0;
    auto chunk = [&](int e0, auto hk) -> bool {
      decltype(load2(0)) g[U];
      TACC va_[U], vb_[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        // entries past this slice's width repeat its last (in bounds) and are not added
        const int e = max(min(e0 + u, wd - 1), 0);
        const int offa = wa > 0 ? ci[oa + max(min(e0 + u, wa - 1), 0)] : 0;
        const int offb = wb > 0 ? ci[ob + max(min(e0 + u, wb - 1), 0)] : 0;
        const int o = useb ? offb : offa;
        if constexpr (PRE_AT_DIAG) {
          if (e0 + u == 0 && o == 0)
            g[u] = pv;  // a leading diagonal: the pair's own operands, already loaded
          else
            g[u] = load2(r0 + o);
        } else {
          g[u] = load2(r0 + o);
        }
        ldval_pair<NT>(vv, (int64_t)e * kSliceRows, va_[u], vb_[u]);
      }
      if constexpr (decltype(hk)::value)
        if (!hook()) return false;
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (e0 + u < wd) {
          const Pair<TACC> o = comb2(g[u]);
          sa += va_[u] * o.x;
          sb += vb_[u] * o.y;
        }
      return true;
    };
    int e0 = 0;
    if constexpr (decltype(first)::value) {
      if (wmax > 0) {
        if (!chunk(0, std::true_type{})) return false;
        e0 = U;
      } else if (!hook()) {
        return false;
      }
    }
    for (; e0 < wmax; e0 += U) chunk(e0, std::false_type{});
    epi2(r0, h0, h1, sa, sb, pv);
    return true;
  };
  int p = w * NW + wv;
  if (p >= npairs) return hook();
  if (!pair(p, std::true_type{})) return false;
  for (p += W * NW; p < npairs; p += W * NW) pair(p, std::false_type{});
  return true;
}

// The two-row walk applies to a sliced-diagonal matrix of at least 2 rows
// placed with two rows per lane.
template <typename TM>
__device__ __forceinline__ bool rows2(const Mat<TM> &M) {
  return M.fmt == FMT_SDIA && M.n >= 2 && M.rpl == 2;
}

template <typename TACC, bool REV = false, bool PRE_AT_DIAG = false, typename TM, typename Pre2, typename Load2,
          typename Comb2, typename Epi2, typename Hook>
__device__ __forceinline__ bool for_rows2(const Mat<TM> &M, int l, int G, Pre2 pre2, Load2 load2, Comb2 comb2,
                                          Epi2 epi2, Hook hook) {
  if (M.temporal) return sdia_rows2<TACC, false, REV, PRE_AT_DIAG>(M, l, G, pre2, load2, comb2, epi2, hook);
  return sdia_rows2<TACC, true, REV, PRE_AT_DIAG>(M, l, G, pre2, load2, comb2, epi2, hook);
}

// Sliced 3x3-block rows: each wave takes whole slices of 21 block rows, one
// lane per row (lane 63 idle); the three lanes of a block row read the same
// block column. 8-byte values are stored column-major within the slice (lane
// 21 s + r for row s of block row r), so each column's values are one
// coalesced load; 4-byte values keep each row's three values contiguous
// (lane 3 r + s), one 12-byte load per lane. Each lane adds its row's three
// products block by block: the CSR order.
template <typename TM>
struct BsrLanes {
  static constexpr bool kColMajor = sizeof(TM) == 8;
  __device__ static int sub(int lane) { return kColMajor ? lane / kBSliceRows : lane % 3; }
  __device__ static int blockrow(int lane) { return kColMajor ? lane % kBSliceRows : lane / 3; }
  // offset of block k's column-j value for this lane, relative to the slice's first block
  __device__ static int64_t at(int lane, int k, int j) {
    return kColMajor ? ((int64_t)k * 3 + j) * (3 * kBSliceRows) + lane
                     : ((int64_t)k * kBSliceRows + lane / 3) * 9 + 3 * (lane % 3) + j;
  }
};

template <typename TACC, bool NT, typename TM, typename Pre, typename Gather, typename Epi>
__device__ __forceinline__ void bsr_rows(const Mat<TM> &M, int l, int G, Pre pre, Gather gather, Epi epi) {
  constexpr int NW = kBlock / 64;
  constexpr int SR = 3 * kBSliceRows;  // rows per slice
  using BL = BsrLanes<TM>;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int W = G >> 3, x = l & 7, w = l >> 3;
  const int s0 = (int)((int64_t)x * M.nblk / 8), s1 = (int)((int64_t)(x + 1) * M.nblk / 8);
  const int sub = BL::sub(lane), r = BL::blockrow(lane);
  for (int c = s0 + w * NW + wv; c < s1; c += W * NW) {
    const int o0 = ro(M.blk)[c], wd = ro(M.blk)[c + 1] - o0;
    const int row = (c * kBSliceRows + r) * 3 + sub;
    const bool has = lane < SR && row < M.n;
    if (!has) continue;
    const RowVals<TACC> pv = pre(row);
    GLOBAL const int32_t *bc = M.ci + (int64_t)o0 * kBSliceRows + r;
    GLOBAL const TM *bv = M.val + (int64_t)o0 * 9 * kBSliceRows;
    TACC sum = 0;
    int k = 0;
    for (; k + 2 <= wd; k += 2) {
      const int32_t c0 = 3 * ldstream<NT>(bc, (int64_t)k * kBSliceRows);
      const int32_t c1 = 3 * ldstream<NT>(bc, (int64_t)(k + 1) * kBSliceRows);
      TACC p[6];
#pragma unroll
      for (int j = 0; j < 3; ++j) p[j] = (TACC)ldval<NT>(bv, BL::at(lane, k, j)) * gather(c0 + j);
#pragma unroll
      for (int j = 0; j < 3; ++j) p[3 + j] = (TACC)ldval<NT>(bv, BL::at(lane, k + 1, j)) * gather(c1 + j);
#pragma unroll
      for (int u = 0; u < 6; ++u) sum += p[u];
    }
    if (k < wd) {
      const int32_t c0 = 3 * ldstream<NT>(bc, (int64_t)k * kBSliceRows);
#pragma unroll
      for (int j = 0; j < 3; ++j) sum += (TACC)ldval<NT>(bv, BL::at(lane, k, j)) * gather(c0 + j);
    }
    epi(row, sum, pv);
  }
}

// All rows of this workgroup (local index l of the system's G workgroups),
// in any layout, with the matrix's load policy.
// DIAG: pre(row).a is the gathered operand at column row (the sliced-diagonal
// walk then reuses it for a diagonal entry).
// UW: loads in flight per lane in sliced rows of more than 4 entries; US:
// products in flight per thread in CSR (stage_products). hook: a workgroup step before the first
// epilogue, after the first products where the layout allows it.
template <typename TACC, int UW, int US, bool NT, bool REV, bool DIAG = false, typename TM, typename Pre,
          typename Gather, typename Epi, typename Hook>
__device__ __forceinline__ bool for_rows_as(const Mat<TM> &M, int l, int G, TACC *lds, Pre pre, Gather gather, Epi epi,
                                            Hook hook) {
  if (M.fmt == FMT_SELL) {
    if constexpr (std::is_same_v<Hook, NoHook>) {
      sell_rows<TACC, UW, NT, REV>(M, l, G, pre, gather, epi);
      return true;
    } else {
      return sell_rows_h<TACC, UW, NT, REV>(M, l, G, pre, gather, epi, hook);
    }
  } else if (M.fmt == FMT_SDIA) {
    if constexpr (std::is_same_v<Hook, NoHook>) {
      sdia_rows<TACC, UW, NT, REV, DIAG>(M, l, G, pre, gather, epi);
      return true;
    } else {
      return sdia_rows_h<TACC, UW, NT, REV>(M, l, G, pre, gather, epi, hook);
    }
  } else if (M.fmt == FMT_BSR3) {
    if (!hook()) return false;
    bsr_rows<TACC, NT>(M, l, G, pre, gather, epi);
    return true;
  } else {
    const Sched sc = sched(M.nblk, l, G);
    int b = sc.first;
    if constexpr (!std::is_same_v<Hook, NoHook>) {
      if (b >= sc.end) return hook();
      if (!stream_block<TACC, US, NT>(M, b, lds, pre, gather, epi, hook)) return false;
      b += sc.stride;
    }
    for (; b < sc.end; b += sc.stride) stream_block<TACC, US, NT>(M, b, lds, pre, gather, epi, NoHook{});
    return true;
  }
}

template <typename TACC, int UW = 4, int US = 0, bool REV = false, bool DIAG = false, typename TM,
          typename Pre, typename Gather, typename Epi>
__device__ __forceinline__ void for_rows(const Mat<TM> &M, int l, int G, TACC *lds, Pre pre, Gather gather, Epi epi) {
  if (M.temporal)
    for_rows_as<TACC, UW, US, false, REV, DIAG>(M, l, G, lds, pre, gather, epi, NoHook{});
  else
    for_rows_as<TACC, UW, US, true, REV, DIAG>(M, l, G, lds, pre, gather, epi, NoHook{});
}

// for_rows with a workgroup step (hook) before the first epilogue: after the
// first slice's products over sliced diagonals, and in the other layouts with
// EARLY (kernels built for one layout), else before the walk. Returns hook's
// result.
template <typename TACC, int UW, int US, bool EARLY, typename TM, typename Pre, typename Gather, typename Epi,
          typename Hook>
__device__ __forceinline__ bool for_rows_h(const Mat<TM> &M, int l, int G, TACC *lds, Pre pre, Gather gather, Epi epi,
                                           Hook hook) {
  if (!EARLY && M.fmt != FMT_SDIA) {
    if (!hook()) return false;
    for_rows<TACC, UW, US>(M, l, G, lds, pre, gather, epi);
    return true;
  }
  if constexpr (EARLY) {
    if (M.temporal) return for_rows_as<TACC, UW, US, false, false>(M, l, G, lds, pre, gather, epi, hook);
    return for_rows_as<TACC, UW, US, true, false>(M, l, G, lds, pre, gather, epi, hook);
  } else {
    if (M.temporal) return sdia_rows_h<TACC, UW, false, false>(M, l, G, pre, gather, epi, hook);
    return sdia_rows_h<TACC, UW, true, false>(M, l, G, pre, gather, epi, hook);
  }
}

// ---- inner products
//
// Every dot product and norm is, up to the bound below, its exact value rounded
// once to FP64, the value that does not depend on how the sum is split over lanes,
// waves and workgroups. Each lane accumulates its products as an unevaluated double-
// double hi + lo (the product's rounding error from an FMA, the additions'
// from TwoSum: Ogita, Rump and Oishi's Dot2); partial sums are combined as
// double-doubles in any order and rounded once at the end. The result is the
// correctly rounded inner product unless the exact value lies within about
// n u^2 sum|a_i b_i| of a rounding boundary (u = 2^-53), which for the sizes
// here is far below one chance in a billion per dot product.
struct Acc {
  double hi, lo;
};

// s + e = a + b exactly, s = fl(a + b) (Knuth's TwoSum; needs no ordering
// of |a|, |b|, and no contraction or reassociation, which the build forbids)
__device__ __forceinline__ void two_sum(double a, double b, double &s, double &e) {
  s = a + b;
  const double bb = s - a;
  e = (a - (s - bb)) + (b - bb);
}

// x += a b: the product's exact error from an FMA (FP64 operands); the
// product of two FP32 values is exact in FP64
__device__ __forceinline__ void acc_prod(Acc &x, double a, double b) {
  const double p = a * b;
  const double pe = __builtin_fma(a, b, -p);
  double s, e;
  two_sum(x.hi, p, s, e);
  x.hi = s;
  x.lo = x.lo + (e + pe);
}
__device__ __forceinline__ void acc_prod(Acc &x, float a, float b) {
  const double p = (double)a * (double)b;
  double s, e;
  two_sum(x.hi, p, s, e);
  x.hi = s;
  x.lo = x.lo + e;
}

// a + b, normalised (hi = fl(hi + lo)): 11 FP64 operations, 9 of them
// dependent. The pair is renormalised by Dekker's Fast2Sum, which gives what
// TwoSum would (three operations more): s is zero, far above t, or a multiple
// of t's last place. Without the renormalisation (8 operations, 6 dependent) the
// low words grow through a tree of sums and their roundings with them: over
// 131,072 lanes the pair's error was twice as large (squares 7.0e-33 of the
// terms' magnitude against 3.6e-33).
__device__ __forceinline__ Acc acc_add(Acc a, Acc b) {
  double s, e;
  two_sum(a.hi, b.hi, s, e);
  const double t = (a.lo + b.lo) + e;
  Acc r;
  r.hi = s + t;
  r.lo = t - (r.hi - s);
  return r;
}

// One DPP move of a double (two 32-bit moves); lanes without a source
// receive 0.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)b, CTRL, 0xF, 0xF, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, true);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
template <int CTRL>
__device__ __forceinline__ Acc acc_dpp(Acc a) {
  return Acc{dpp_f64<CTRL>(a.hi), dpp_f64<CTRL>(a.lo)};
}

// Wave total of a double-double by DPP row operations, with no LDS traffic,
// in lane 63. The two quad exchanges, the half-row mirror and the row mirror
// leave each 16-lane row's total in all of its lanes. Two row broadcasts then
// carry rows 0 to 2 into row 3: lane 15 of each row into the next row (row 1
// holds rows 0 + 1, row 3 rows 2 + 3), then lane 31 into rows 2 and 3. What
// the other rows hold after that is not used.
__device__ __forceinline__ Acc wave_total(Acc v) {
  v = acc_add(v, acc_dpp<0xB1>(v));   // quad_perm [1,0,3,2]
  v = acc_add(v, acc_dpp<0x4E>(v));   // quad_perm [2,3,0,1]
  v = acc_add(v, acc_dpp<0x141>(v));  // row_half_mirror
  v = acc_add(v, acc_dpp<0x140>(v));  // row_mirror
  v = acc_add(v, acc_dpp<0x142>(v));  // row_bcast:15
  v = acc_add(v, acc_dpp<0x143>(v));  // row_bcast:31
  return v;
}

// Wave totals of two double-doubles at once: a in lane 31, b in lane 63. One
// exchange of wave halves leaves 32 partial sums of a in the lower half and 32
// of b in the upper, so the remaining steps serve both (6 additions, not 12).
__device__ __forceinline__ void swap_halves(double &a, double &b) {
  const uint64_t x = (uint64_t)__double_as_longlong(a), y = (uint64_t)__double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
  a = __longlong_as_double((long long)(((uint64_t)hi[0] << 32) | lo[0]));
  b = __longlong_as_double((long long)(((uint64_t)hi[1] << 32) | lo[1]));
}
__device__ __forceinline__ Acc wave_total2(Acc a, Acc b) {
  swap_halves(a.hi, b.hi);
  swap_halves(a.lo, b.lo);
  Acc v = acc_add(a, b);
  v = acc_add(v, acc_dpp<0xB1>(v));
  v = acc_add(v, acc_dpp<0x4E>(v));
  v = acc_add(v, acc_dpp<0x141>(v));
  v = acc_add(v, acc_dpp<0x140>(v));
  v = acc_add(v, acc_dpp<0x142>(v));
  return v;
}

// The total of each group of N adjacent lanes (a power of two up to 8), in all of
// the group.
template <int N>
__device__ __forceinline__ Acc lanes_total(Acc v) {
  static_assert(N == 1 || N == 2 || N == 4 || N == 8, "lanes");
  if constexpr (N >= 2) v = acc_add(v, acc_dpp<0xB1>(v));
  if constexpr (N >= 4) v = acc_add(v, acc_dpp<0x4E>(v));
  if constexpr (N >= 8) v = acc_add(v, acc_dpp<0x141>(v));
  return v;
}

// A lane's double, in every lane.
__device__ __forceinline__ double readlane_f64(double v, int lane) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, lane), hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), lane);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Each wave's totals of the NV values into sh[j NW + wave].
template <int NV>
__device__ __forceinline__ void put_wave_totals(const Acc (&v)[NV], Acc *sh) {
  static_assert(NV == 1 || NV == 2, "values");
  constexpr int NW = kBlock / 64;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if constexpr (NV == 1) {
    const Acc t = wave_total(v[0]);
    if (lane == 63) sh[w] = t;
  } else {
    const Acc t = wave_total2(v[0], v[1]);
    if ((lane & 31) == 31) sh[(lane >> 5) * NW + w] = t;
  }
}

// The wave totals in sh[0, NW) added pairwise.
__device__ __forceinline__ Acc add_waves(const Acc *sh) {
  constexpr int NW = kBlock / 64;
  Acc a[NW];
#pragma unroll
  for (int q = 0; q < NW; ++q) a[q] = sh[q];
#pragma unroll
  for (int h = NW / 2; h >= 1; h /= 2)
#pragma unroll
    for (int q = 0; q < h; ++q) a[q] = acc_add(a[q], a[q + h]);
  return a[0];
}

// Workgroup total of each value, in thread 0; sh[0, NV NW).
template <int NV>
__device__ __forceinline__ void block_sum(Acc (&v)[NV], Acc *sh) {
  constexpr int NW = kBlock / 64;
  put_wave_totals<NV>(v, sh);
  __syncthreads();
  if (threadIdx.x == 0)
#pragma unroll
    for (int j = 0; j < NV; ++j) v[j] = add_waves(sh + j * NW);
  __syncthreads();
}

// Write this workgroup's partial sums: value j's hi at p[2j G + L], its lo at
// p[(2j + 1) G + L] (kAccWords doubles per partial).
template <int NV>
__device__ __forceinline__ void put_partials(Acc (&v)[NV], GLOBAL double *p, int L, int G, Acc *sh) {
  block_sum<NV>(v, sh);
  if (threadIdx.x == 0)
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      p[(int64_t)(2 * j) * G + L] = v[j].hi;
      p[(int64_t)(2 * j + 1) * G + L] = v[j].lo;
    }
}

// Total of the P partials of each value; every thread gets the totals,
// rounded once to FP64. load_partials adds this thread's share (no barrier,
// so a kernel can issue it before it reads its state); reduce_partials
// finishes the sums.
template <int NV>
__device__ __forceinline__ void load_partials(GLOBAL const double *__restrict__ p, int P, Acc (&acc)[NV]) {
#pragma unroll
  for (int j = 0; j < NV; ++j) acc[j] = Acc{0.0, 0.0};
#pragma unroll 4
  for (int k = threadIdx.x; k < P; k += kBlock)
#pragma unroll
    for (int j = 0; j < NV; ++j) acc[j] = acc_add(acc[j], Acc{p[(int64_t)(2 * j) * P + k], p[(int64_t)(2 * j + 1) * P + k]});
}

// A value every lane holds alike, as a wave-uniform (scalar) value.
__device__ __forceinline__ double uniform(double v) {
  const uint64_t b = __double_as_longlong(v);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b), hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// The wave totals meet in LDS after one barrier, and each wave adds them
// across its lanes: two additions in sequence for both values at once (with
// every lane adding all of them, a solve of 2025 rows by the one-workgroup
// stencil solver takes 385 us against 354). They sit in sh[2 NW, 2 NW + NV NW),
// apart from block_sum's slots, so that a block_sum later in the kernel cannot
// overwrite them while a slower wave still reads them; callers put a barrier
// between two calls.
template <int NV>
__device__ __forceinline__ void reduce_partials(Acc (&acc)[NV], double (&out)[NV], Acc *sh) {
  static_assert(NV <= 2, "reduction slots");
  constexpr int NW = kBlock / 64;
  Acc *shr = sh + 2 * NW;
  put_wave_totals<NV>(acc, shr);
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const Acc a = lanes_total<NW>(shr[(NV == 2 ? (lane >> 5) * NW : 0) + (lane & (NW - 1))]);
  out[0] = readlane_f64(a.hi + a.lo, 0);
  if constexpr (NV == 2) out[1] = readlane_f64(a.hi + a.lo, 32);
}

template <int NV>
__device__ __forceinline__ void sum_partials(GLOBAL const double *__restrict__ p, int P, double (&out)[NV],
                                             Acc *sh) {
  Acc acc[NV];
  load_partials<NV>(p, P, acc);
  reduce_partials<NV>(acc, out, sh);
}

// The system a workgroup works for and its local index there. A launch over
// one system (map = nullptr) takes the system's record as a kernel argument;
// a launch over many looks its (system, local workgroup) up in the map and
// the record in the directory. Both of those are dependent loads that miss
// every cache after a kernel boundary (the first touch comes from memory), in
// front of everything else a workgroup does: the argument takes two memory
// round trips off each launch of a single solve.
struct Work {
  SysDev D;
  int l;
};
__device__ __forceinline__ Work work_of(const SysDev *__restrict__ dir, const int2 *__restrict__ map,
                                        const SysDev &one) {
  Work w;
  if (map) {
    const int2 m = map[blockIdx.x];
    w.D = dir[m.x];
    w.l = m.y;
  } else {
    w.D = one;
    w.l = (int)blockIdx.x;
  }
  return w;
}

// Tells the host how far a solve has come: 2 iter + done into a word of
// page-locked host memory, from the thread that publishes the state. A copy of
// the state and an event after every graph of ten iterations took 18 us of the
// stream (gaps of 8.5 and 5.6 us around a 4 us copy), 1.8 us per iteration.
__device__ __forceinline__ void report_progress(uint64_t *report, int32_t iter, int32_t done) {
  if (report)
    __hip_atomic_store(report, 2 * (uint64_t)(uint32_t)iter + (done ? 1 : 0), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
}

// Rows [l n / G, (l+1) n / G) of a system: local workgroup l's share of
// elementwise work over G workgroups.
__device__ __forceinline__ void ew_rows(int n, int l, int G, int64_t &i0, int64_t &i1) {
  i0 = (int64_t)l * n / G;
  i1 = (int64_t)(l + 1) * n / G;
}

}  // namespace pcgk
