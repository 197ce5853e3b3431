// The iteration kernels (iter.h) built for one layout each, for launches over a
// single system in CSR row blocks, sliced ELL or 3x3 blocks. Stencils go to their
// own kernels, and sliced diagonals that those cannot hold to the ones built for
// every layout.
// Built with floating-point contraction off, like every kernel here.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include "iter.h"

namespace pcgk {

#define PCG_SINGLE(kern, grid, ...)                                                             \
  do {                                                                                          \
    if (e0 || e1)                                                                               \
      hipExtLaunchKernelGGL(kern, dim3(grid), dim3(kBlock), 0, s, e0, e1, 0, __VA_ARGS__);      \
    else                                                                                        \
      hipLaunchKernelGGL(kern, dim3(grid), dim3(kBlock), 0, s, __VA_ARGS__);                    \
  } while (0)

#define PCG_SINGLE_FMT(fmt_, FMT, ...)                                     \
  switch (fmt_) {                                                          \
    case FMT_CSR: { constexpr int FMT = FMT_CSR; __VA_ARGS__; break; }     \
    case FMT_SELL: { constexpr int FMT = FMT_SELL; __VA_ARGS__; break; }   \
    case FMT_BSR3: { constexpr int FMT = FMT_BSR3; __VA_ARGS__; break; }   \
    default: return hipErrorInvalidValue;                                  \
  }

// The storage types a context may have: FP32 vectors go with a G of FP32 or less.
#define PCG_SINGLE_TYPES(ty, TV, TG, ...)                                                                  \
  if ((ty).vec == F64 && (ty).g == F64) { using TV = double; using TG = double; __VA_ARGS__; }             \
  else if ((ty).vec == F64 && (ty).g == F32) { using TV = double; using TG = float; __VA_ARGS__; }         \
  else if ((ty).vec == F64 && (ty).g == BF16) { using TV = double; using TG = bf16_t; __VA_ARGS__; }       \
  else if ((ty).vec == F64 && (ty).g == F16) { using TV = double; using TG = _Float16; __VA_ARGS__; }      \
  else if ((ty).vec == F32 && (ty).g == F32) { using TV = float; using TG = float; __VA_ARGS__; }          \
  else if ((ty).vec == F32 && (ty).g == BF16) { using TV = float; using TG = bf16_t; __VA_ARGS__; }        \
  else if ((ty).vec == F32 && (ty).g == F16) { using TV = float; using TG = _Float16; __VA_ARGS__; }       \
  else return hipErrorInvalidValue;

hipError_t launch_one_A(const Types &ty, const LaunchSet &L, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  const bool u4 = L.uw_a == 4;
  PCG_SINGLE_FMT(L.one->A.fmt, FMT, {
    if (ty.vec == F64 && ty.a == F64) {
      if (u4)
        PCG_SINGLE((k_iter_A<double, double, 4, FMT>), L.nA, L.dir, nullptr, *L.one);
      else
        PCG_SINGLE((k_iter_A<double, double, 8, FMT>), L.nA, L.dir, nullptr, *L.one);
    } else if (ty.vec == F32 && ty.a == F32) {
      if (u4)
        PCG_SINGLE((k_iter_A<float, float, 4, FMT>), L.nA, L.dir, nullptr, *L.one);
      else
        PCG_SINGLE((k_iter_A<float, float, 8, FMT>), L.nA, L.dir, nullptr, *L.one);
    } else {
      return hipErrorInvalidValue;
    }
  });
  return hipGetLastError();
}

hipError_t launch_one_GT(const Types &ty, const LaunchSet &L, int mode, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  PCG_SINGLE_FMT(L.one->GT.fmt, FMT, {
    PCG_SINGLE_TYPES(ty, TV, TG, {
      PCG_SINGLE((k_iter_GT<TV, TG, FMT>), L.nGT, L.dir, nullptr, *L.one, mode);
    })
  });
  return hipGetLastError();
}

hipError_t launch_one_G(const Types &ty, const LaunchSet &L, bool has_eps, int mode, hipStream_t s, hipEvent_t e0,
                        hipEvent_t e1, uint64_t *report) {
  PCG_SINGLE_FMT(L.one->G.fmt, FMT, {
    PCG_SINGLE_TYPES(ty, TV, TG, {
      if (has_eps)
        PCG_SINGLE((k_iter_G<TV, TG, true, FMT>), L.nG, L.dir, nullptr, *L.one, mode, report);
      else
        PCG_SINGLE((k_iter_G<TV, TG, false, FMT>), L.nG, L.dir, nullptr, *L.one, mode, report);
    })
  });
  return hipGetLastError();
}

}  // namespace pcgk
