"""Register budget of the kernels beside the iteration kernels' own file
(compiled for gfx950 on the host, no GPU needed): none spills to scratch
memory, and the stencil iteration kernels keep the four waves per SIMD that
their grid fills, the products eight."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2510_27517_amd", "csrc")


SOURCES = ["wg.hip", "dia.hip", "wgs.hip", "products.hip"]


def _compile(source, out):
    from paper_2510_27517_amd import build

    cmd = [build.HIPCC, *build.COMMON, *build.DEVICE, "-Rpass-analysis=kernel-resource-usage", "-c",
           os.path.join(CSRC, source), "-o", str(out / (source + ".o"))]
    return subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)


@pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="hipcc not installed")
def test_no_spills(tmp_path):
    least = [(r"k_dia_(A|GT|G)I", 4), (r"k_(spmv|spmm|spmm_loss)I", 8)]
    with ThreadPoolExecutor(max_workers=4) as pool:
        runs = list(pool.map(lambda s: _compile(s, tmp_path), SOURCES))
    for source, r in zip(SOURCES, runs):
        assert r.returncode == 0, r.stdout[-2000:]
        names = re.findall(r"Function Name: (\S+)", r.stdout)
        scratch = [int(x) for x in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stdout)]
        waves = [int(x) for x in re.findall(r"Occupancy \[waves/SIMD\]: (\d+)", r.stdout)]
        assert names and len(names) == len(scratch) == len(waves), source
        assert not [(k, s) for k, s in zip(names, scratch) if s]
        assert not [(k, w) for k, w in zip(names, waves) for p, m in least if re.search(p, k) and w < m]
