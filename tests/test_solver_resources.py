"""Register budget of the kernels beside the iteration kernels' own file
(compiled for gfx950 on the host, no GPU needed): none spills to scratch
memory, and the stencil iteration kernels keep the four waves per SIMD that
their grid fills."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2510_27517_amd", "csrc")


@pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="hipcc not installed")
@pytest.mark.parametrize("source", ["wg.hip", "dia.hip", "wgs.hip"])
def test_no_spills(tmp_path, source):
    from paper_2510_27517_amd import build

    cmd = [build.HIPCC, *build.COMMON, *build.DEVICE, "-Rpass-analysis=kernel-resource-usage", "-c",
           os.path.join(CSRC, source), "-o", str(tmp_path / "k.o")]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-2000:]
    names = re.findall(r"Function Name: (\S+)", r.stdout)
    scratch = [int(x) for x in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stdout)]
    waves = [int(x) for x in re.findall(r"Occupancy \[waves/SIMD\]: (\d+)", r.stdout)]
    assert names and len(names) == len(scratch) == len(waves)
    assert not [(k, s) for k, s in zip(names, scratch) if s]
    assert not [(k, w) for k, w in zip(names, waves) if re.search(r"k_dia_(A|GT|G)I", k) and w < 4]
