"""A file of autotuner choices written before stencil storage existed does
not switch that storage off: its entries (signatures without a version) are
searched again, and only entries of this version are applied."""
import json
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = """
import json, sys
sys.path.insert(0, sys.argv[1])
from paper_2510_27517_amd import inputs, pcg
A = inputs.poisson(3, 64, 1.0, 11)
with pcg.Solver(pcg.default_config()) as s:
    s.set_matrix(A)
    s.build_precond(pcg.G_FSAI)
    t = s.autotune(10)
    r = s.solve(inputs.rhs(A.n, 1), tol=1e-8, maxit=5000)
print(json.dumps(dict(t, iters=r.iters, bytes=r.bytes_per_iter)))
"""


def _run(cache):
    r = subprocess.run([sys.executable, "-c", PROGRAM, ROOT], env=dict(os.environ, PCG_TUNE_CACHE=str(cache)),
                       stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads(r.stdout.splitlines()[-1])


def test_entries_of_an_earlier_version(gpu_lib, tmp_path):
    pcg = gpu_lib
    first = _run(tmp_path / "new.txt")
    assert first["candidates"] > 0
    line = (tmp_path / "new.txt").read_text().split()
    again = _run(tmp_path / "new.txt")
    assert again["candidates"] == 0 and again["bytes"] == first["bytes"]
    old = [line[0].split("_v")[0], str(pcg.LAYOUT_CSR), str(pcg.LAYOUT_CSR)] + line[3:]
    (tmp_path / "old.txt").write_text(" ".join(old) + "\n")
    # searched, not applied (what the search picks depends on its timings)
    after = _run(tmp_path / "old.txt")
    assert after["candidates"] > 0 and after["iters"] == first["iters"]
