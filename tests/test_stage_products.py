"""Staging of a CSR row block's products: every entry of the block once and
nothing beside it, also where the nonzeros' numbers end just below 2^31. The
kernels' own loop, compiled for the host and run thread by thread with loads
that only record their index."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = """
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <vector>
#define __device__
#define __forceinline__ inline
using std::min;
constexpr int kBlock = 256;
struct Id { unsigned x; } threadIdx;
static int64_t lo, hi;
static std::vector<int> seen;
struct Ptr {};
static void check(int64_t k) {
  if (k < lo || k >= hi) {
    std::printf("entry %lld outside [%lld, %lld)\\n", (long long)k, (long long)lo, (long long)hi);
    std::exit(2);
  }
}
template <bool NT> double ldval(Ptr, int64_t k) { check(k); return 1.0; }
template <bool NT> int32_t ldstream(Ptr, int64_t k) { check(k); return 0; }
template <typename TM> struct Mat { Ptr val, ci; };
struct Lds {
  struct Slot { Slot &operator=(double) { return *this; } };
  Slot s;
  Slot &operator[](int64_t k) {
    if (k < 0 || k >= hi - lo) { std::printf("slot %lld\\n", (long long)k); std::exit(3); }
    ++seen[k];
    return s;
  }
};
@LOOP@
template <int U> void run(int64_t c0, int64_t c1) {
  lo = c0, hi = c1;
  seen.assign(c1 - c0, 0);
  Lds lds;
  for (unsigned t = 0; t < kBlock; ++t) {
    threadIdx.x = t;
    stage_products<double, U, true>(Mat<double>{}, (int)c0, (int)c1, lds, [](int) { return 1.0; });
  }
  for (int k : seen)
    if (k != 1) { std::printf("an entry staged %d times\\n", k); std::exit(4); }
}
int main() {
  const int64_t top = INT32_MAX;
  for (int64_t c1 : {int64_t(5000), top - 4096, top - 2048, top - 255, top - 1, top})
    for (int64_t len : {0, 1, 255, 256, 257, 2047, 2048, 4096}) {
      run<0>(c1 - len, c1);
      run<1>(c1 - len, c1);
      run<8>(c1 - len, c1);
    }
  return 0;
}
"""


def test_every_entry_once(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not installed")
    src = open(os.path.join(ROOT, "paper_2510_27517_amd", "csrc", "device.h")).read()
    at = src.rindex("template", 0, src.index("void stage_products("))
    loop = src[at:src.index("\n}\n", at) + 3]
    loop = loop.replace("TACC *lds", "Lds &lds")  # so that each store is seen
    (tmp_path / "h.cpp").write_text(HARNESS.replace("@LOOP@", loop))
    subprocess.run([gxx, "-O1", "-fwrapv", "-std=c++17", "-Wno-unknown-pragmas", "-o", str(tmp_path / "h"),
                    str(tmp_path / "h.cpp")], check=True)
    r = subprocess.run([str(tmp_path / "h")], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, timeout=60)
    assert r.returncode == 0, r.stdout
