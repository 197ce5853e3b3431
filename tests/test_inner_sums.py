"""The double-double additions of the kernels' inner products, compiled for
the host from the kernels' own header: sums stay normalised, and a tree of them
is as accurate as one that renormalises every sum by TwoSum."""
import ctypes
import os
import shutil
import subprocess
from fractions import Fraction

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = """
#define __device__
#define __forceinline__ inline
%s
extern "C" void tree(double *hi, double *lo, int n, int full) {  // n a power of two; the sum to [0]
  for (int h = n / 2; h >= 1; h /= 2)
    for (int i = 0; i < h; ++i) {
      Acc r;
      if (full) {
        double s, e;
        two_sum(hi[i], hi[i + h], s, e);
        const double t = (lo[i] + lo[i + h]) + e;
        two_sum(s, t, r.hi, r.lo);
      } else {
        r = acc_add(Acc{hi[i], lo[i]}, Acc{hi[i + h], lo[i + h]});
      }
      hi[i] = r.hi;
      lo[i] = r.lo;
    }
}
extern "C" void products(const double *a, const double *b, int n, int m, double *hi, double *lo) {
  for (int i = 0; i < n; ++i) {
    Acc x{0.0, 0.0};
    for (int k = 0; k < m; ++k) acc_prod(x, a[i * m + k], b[i * m + k]);
    hi[i] = x.hi;
    lo[i] = x.lo;
  }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not installed")
    src = open(os.path.join(ROOT, "paper_2510_27517_amd", "csrc", "device.h")).read()
    part = src[src.index("struct Acc {"):src.index("// One DPP move of a double")]
    d = tmp_path_factory.mktemp("sums")
    (d / "sums.cpp").write_text(HARNESS % part)
    subprocess.run([gxx, "-O2", "-ffp-contract=off", "-shared", "-fPIC", "-o", str(d / "sums.so"),
                    str(d / "sums.cpp")], check=True)
    return ctypes.CDLL(str(d / "sums.so"))


def _operands(kind, n, m, rng):
    a = rng.standard_normal((n, m))
    if kind == "squares":
        return a, a.copy()
    if kind == "cancelling":
        return a, rng.standard_normal((n, m))
    if kind == "scales":
        return a * 10.0 ** rng.uniform(-8, 8, (n, m)), rng.standard_normal((n, m))
    b = rng.standard_normal((n, m))  # each lane's second half cancels its first nearly
    a[:, m // 2:], b[:, m // 2:] = -a[:, :m // 2], b[:, :m // 2] * (1.0 + 1e-15)
    return a, b


@pytest.mark.parametrize("kind", ["squares", "cancelling", "scales", "nearly_zero"])
def test_tree_of_sums(lib, kind):
    n, m = 8192, 6
    err = {0: [], 1: []}
    for seed in range(6):
        a, b = _operands(kind, n, m, np.random.default_rng(seed))
        hi, lo = np.empty(n), np.empty(n)
        ptr = lambda v: v.ctypes.data_as(ctypes.c_void_p)
        lib.products(ptr(a), ptr(b), n, m, ptr(hi), ptr(lo))
        exact = sum((Fraction(float(v)) for v in np.concatenate([hi, lo])), Fraction(0))
        size = float(np.abs(a * b).sum())
        for full in (0, 1):
            h, l = hi.copy(), lo.copy()
            lib.tree(ptr(h), ptr(l), n, full)
            assert h[0] + l[0] == h[0]
            err[full].append(float(abs(Fraction(h[0]) + Fraction(l[0]) - exact)) / size)
    # the same to the last bit but for lanes whose sum cancelled
    assert sum(err[0]) <= 1.02 * sum(err[1])
