"""Register budget of the single system's kernels built for one layout each
(compiled for gfx950 on the host, no GPU needed): none spills to scratch memory,
the A-kernel keeps its eight waves per SIMD and the others the four that their
grid fills."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2510_27517_amd", "csrc")


@pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="hipcc not installed")
def test_no_spills(tmp_path):
    from paper_2510_27517_amd import build

    cmd = [build.HIPCC, *build.COMMON, *build.DEVICE, "-Rpass-analysis=kernel-resource-usage", "-c",
           os.path.join(CSRC, "single.hip"), "-o", str(tmp_path / "single.o")]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-2000:]
    names = re.findall(r"Function Name: (\S+)", r.stdout)
    scratch = [int(x) for x in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stdout)]
    waves = [int(x) for x in re.findall(r"Occupancy \[waves/SIMD\]: (\d+)", r.stdout)]
    assert len(names) == len(scratch) == len(waves)
    for kernel, least in ((r"k_iter_AI", 8), (r"k_iter_GTI", 4), (r"k_iter_GI", 4)):
        at = [k for k, name in enumerate(names) if re.search(kernel, name)]
        assert at and not [names[k] for k in at if scratch[k] or waves[k] < least]
