"""Conversion of a matrix's values to their storage type (host code, compiled
here): each value as rounded by itself, at the speed of a plain loop."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2510_27517_amd", "csrc")

HARNESS = """
#include <chrono>
#include "host.h"
using namespace pcgh;
extern "C" void cast(const double *v, int64_t n, int dt, double scale, uint8_t *out, int64_t bytes) {
  Bytes b;
  cast_values(v, n, dt, scale, b);
  std::copy_n(b.data(), bytes, out);
}
extern "C" void times(const double *v, int64_t n, double *ms) {  // library, a plain loop; FP64, then FP32
  Bytes b;
  for (int k = 0; k < 4; ++k) ms[k] = 1e30;
  for (int rep = 0; rep < 25; ++rep)
    for (int k = 0; k < 4; ++k) {
      const auto t0 = std::chrono::steady_clock::now();
      if (k % 2 == 0) {
        cast_values(v, n, k / 2, 1.0, b);
      } else {
        b.resize((size_t)n * (k == 1 ? 8 : 4));
        if (k == 1)
          for (int64_t i = 0; i < n; ++i) ((double *)b.data())[i] = v[i] * 1.0;
        else
          for (int64_t i = 0; i < n; ++i) ((float *)b.data())[i] = (float)(v[i] * 1.0);
      }
      ms[k] = std::min(ms[k], std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count());
    }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    from paper_2510_27517_amd import build

    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc not installed")
    d = tmp_path_factory.mktemp("cast")
    (d / "h.cpp").write_text(HARNESS)
    inc = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(build.HIPCC))), "include")
    subprocess.run([build.HIPCC, *build.COMMON, "-x", "c++", "-D__HIP_PLATFORM_AMD__", f"-I{inc}", "-shared",
                    str(d / "h.cpp"), os.path.join(CSRC, "host.cpp"), "-o", str(d / "h.so"), "-lpthread"], check=True)
    return ctypes.CDLL(str(d / "h.so"))


def _p(a):
    return a.ctypes.data_as(ctypes.c_void_p)


@pytest.mark.parametrize("n", [0, 1, 7, 1000])
@pytest.mark.parametrize("dt", ["f64", "f32", "bf16", "f16"])
def test_values(lib, n, dt):
    import torch

    v = np.random.default_rng(n).standard_normal(n)
    out = np.zeros(n, {"f64": np.float64, "f32": np.float32}.get(dt, np.uint16))
    scale = 0.37
    lib.cast(_p(v), ctypes.c_int64(n), ["f64", "f32", "bf16", "f16"].index(dt), ctypes.c_double(scale), _p(out),
             ctypes.c_int64(out.nbytes))
    want = v * scale
    if dt == "f32":
        want = want.astype(np.float32)
    elif dt == "f16":
        want = want.astype(np.float16).view(np.uint16)
    elif dt == "bf16":  # torch goes through FP32: the same but on ties
        want = torch.from_numpy(want).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)
    assert np.array_equal(out, want)


# values that stay in the cache: a call per value with a switch inside takes five
# to seven times as long as the loop
def test_time(lib):
    v = np.random.default_rng(1).standard_normal(100_000)
    ms = np.zeros(4)
    lib.times(_p(v), ctypes.c_int64(v.size), _p(ms))
    assert ms[0] <= 2.5 * ms[1] and ms[2] <= 2.5 * ms[3], ms
