"""Which solver a small system of few diagonals takes, on both sides of each
bound. A system that the one-workgroup stencil solver takes builds no stencil
storage for the iteration kernels, so its bytes per iteration are the sliced
diagonals'; one that it leaves to them reports the stencil storage's."""
import numpy as np
import pytest

from paper_2510_27517_amd import inputs
from test_gpu_stencil import _banded

pytestmark = pytest.mark.gpu

F32 = dict(vec_dtype="f32", a_dtype="f32", g_dtype="f32")
SEVEN, FIVE = (1, 9, 100), (1, 40)


def _one_workgroup(pcg, A, **kw):
    b = inputs.rhs(A.n, 2)

    def solve(**more):
        with pcg.Solver(pcg.default_config(**{**kw, **more})) as s:
            s.set_matrix(A)
            s.build_precond(pcg.G_FSAI)
            return s.solve(b, tol=1e-6, maxit=400)

    chosen, three, general = solve(), solve(wg_max_n=-1), solve(wg_max_n=-1, layout="sdia")
    assert chosen.iters == three.iters and np.array_equal(chosen.x, three.x)
    if three.bytes_per_iter == general.bytes_per_iter:
        return None  # diagonals too short for stencil storage: the choice does not show
    assert chosen.bytes_per_iter in (three.bytes_per_iter, general.bytes_per_iter)
    return chosen.bytes_per_iter == general.bytes_per_iter


@pytest.mark.parametrize("offsets,n,types,taken", [
    (SEVEN, 1024, {}, True), (SEVEN, 1025, {}, False),      # FP64 of more than 5 and 3 diagonals
    (FIVE, 2048, {}, True), (FIVE, 2049, {}, False),
    (SEVEN, 2048, F32, True), (SEVEN, 2049, F32, False),
    ((1, 9, 50, 100), 700, {}, False),                       # nine diagonals of A
])
def test_rows_and_diagonals(gpu_lib, offsets, n, types, taken):
    assert _one_workgroup(gpu_lib, _banded(n, offsets, 3), **types) is taken


def test_configured_bound(gpu_lib):
    A = _banded(900, FIVE, 3)
    assert _one_workgroup(gpu_lib, A, wg_max_n=900) is True
    assert _one_workgroup(gpu_lib, A, wg_max_n=899) is False


@pytest.mark.parametrize("types", [{}, F32], ids=["f64", "f32"])
@pytest.mark.parametrize("far", [400, 1000, 2000, 2047])
def test_far_diagonal(gpu_lib, far, types):
    """A diagonal far out: three vectors with its distance on either side, up to
    147 KB of a workgroup's LDS."""
    assert _one_workgroup(gpu_lib, _banded(2048, (far,), 3), **types) in (True, None)
