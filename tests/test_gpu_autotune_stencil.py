"""The autotuner on a system that runs over stencil storage."""
import numpy as np
import pytest

from paper_2510_27517_amd import inputs

pytestmark = pytest.mark.gpu


def test_times_every_policy_once_and_no_knob_without_effect(gpu_lib):
    """Candidates: the automatic choice, three layouts of A with three of G,
    two grids, and three load policies, those that differ from the plan's: A
    alone, G alone, both or none of them. The plan of the general kernels (A
    alone in this cache size) is not the stencil's (both)."""
    pcg = gpu_lib
    A = inputs.poisson(3, 64, 1.0, 11)
    b = inputs.rhs(A.n, 11)
    with pcg.Solver(pcg.default_config(cache_mb=40)) as s:
        s.set_matrix(A)
        s.build_precond(pcg.G_FSAI)
        want = s.solve(b, tol=1e-8, maxit=5000)
        t = s.autotune(10)
        got = s.solve(b, tol=1e-8, maxit=5000)
    if t["layout_a"] == t["layout_g"] == pcg.LAYOUT_AUTO:
        assert t["candidates"] == 1 + 3 * 3 + 2 + 3, t
        assert t["temporal"] in (0, 1, 6, 7)
    else:  # a layout asked for was timed faster: no stencil storage, every subset and both knobs
        assert t["candidates"] == 1 + 3 * 3 + 2 + 7 + 2, t
    assert got.iters == want.iters and np.array_equal(got.x, want.x)
