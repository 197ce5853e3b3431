"""Host work in parts: a process whose CPUs change between two counts of them
(another thread or a manager sets its affinity) gets the same layout."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2510_27517_amd", "csrc")

# the C library's call replaced by one whose answer grows (or shrinks) after `first`
HARNESS = """
#include <cstdio>
#include <cstdlib>
#include <sched.h>
#include "host.h"
static int calls, first, before, after;
extern "C" int sched_getaffinity(pid_t, size_t, cpu_set_t *cs) {
  CPU_ZERO(cs);
  const int cpus = calls++ < first ? before : after;
  for (int k = 0; k < cpus; ++k) CPU_SET(k, cs);
  return 0;
}
int main(int argc, char **argv) {
  first = atoi(argv[1]), before = atoi(argv[2]), after = atoi(argv[3]);
  const int n = 1 << 17;
  std::vector<int32_t> rp(1, 0), ci, so, offs, so1, offs1;
  for (int i = 0; i < n; ++i) {
    for (int o : {-300, -1, 0, 1, 300})
      if (i + o >= 0 && i + o < n) ci.push_back(i + o);
    rp.push_back((int32_t)ci.size());
  }
  const bool ok = pcgh::sdia_pattern(n, rp.data(), ci.data(), INT64_MAX, so, offs, 0);
  const bool ok1 = pcgh::sdia_pattern(n, rp.data(), ci.data(), INT64_MAX, so1, offs1, 1);
  std::printf("%d\\n", calls);
  return ok && ok1 && so == so1 && offs == offs1 ? 0 : 1;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    from paper_2510_27517_amd import build

    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc not installed")
    d = tmp_path_factory.mktemp("parts")
    (d / "h.cpp").write_text(HARNESS)
    inc = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(build.HIPCC))), "include")
    subprocess.run([build.HIPCC, *build.COMMON, "-x", "c++", "-D__HIP_PLATFORM_AMD__", f"-I{inc}", str(d / "h.cpp"),
                    os.path.join(CSRC, "host.cpp"), "-o", str(d / "h"), "-lpthread"], check=True)
    return str(d / "h")


@pytest.mark.parametrize("before,after", [(1, 8), (2, 8), (8, 1), (8, 8)])
def test_affinity_changes(program, before, after):
    r = subprocess.run([program, "1", str(before), str(after)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                       timeout=60)
    assert r.returncode == 0 and int(r.stdout) >= 1, (r.returncode, r.stdout)
