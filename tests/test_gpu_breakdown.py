"""What a solve that breaks down reports: the residual of the iterate it
leaves, the same whichever solver ran."""
import types

import numpy as np
import pytest

from paper_2510_27517_amd import inputs
from paper_2510_27517_amd.inputs import CSR

pytestmark = pytest.mark.gpu

TYPES = {"f64": {}, "f32_bf16": dict(vec_dtype="f32", a_dtype="f32", g_dtype="bf16")}


def _indefinite(side):
    """A 2D grid's matrix shifted past its lowest eigenvalue: CG goes on for
    some iterations before d^T A d <= 0."""
    import scipy.sparse as sp
    from scipy.sparse.linalg import eigsh

    A = inputs.poisson(2, side, 1.0, 7).to_scipy().tocsr()
    low = eigsh(A, k=1, sigma=0.0, return_eigenvectors=False)[0]
    A = (A - 1.5 * low * sp.identity(A.shape[0])).tocsr()
    A.sort_indices()
    return CSR.from_scipy(A)


def _solve(pcg, A, b, device, **kw):
    with pcg.Solver(pcg.default_config(**kw)) as s:
        s.set_matrix(A)
        s.build_precond(pcg.G_JACOBI)
        if device:
            import torch

            r = s.solve(torch.from_numpy(b).cuda(), tol=1e-12, maxit=400, allow_failure=True)
            r.x = r.x.cpu().numpy()
            return r
        return s.solve(b, tol=1e-12, maxit=400, allow_failure=True)


def _batch(pcg, A, b, **kw):
    """Two copies of the system solved as a batch, the first one's result."""
    with pcg.Solver(pcg.default_config(mem_budget_mb=64, **kw)) as s:
        out = s.solve_batch([dict(A=A, b=b, g_kind=pcg.G_JACOBI, tol=1e-12, maxit=400)] * 2)
    x, r = out[0]
    return types.SimpleNamespace(x=x, **r)


def _check(A, b, got, want, fp64):
    assert got.status == want.status < 0 and got.iters == want.iters > 0
    assert np.array_equal(got.x, want.x)
    assert got.relres_true == want.relres_true and got.relres_rec == want.relres_rec
    # the residual is of the size of b: its sums of a few products err by far less
    if fp64:
        res = np.linalg.norm(b - A.to_scipy() @ got.x) / np.linalg.norm(b)
        assert abs(got.relres_true - res) <= 1e-10 * res


# 8^2 rows: one wave; 22^2 and 23^2: either side of 512 rows; 45^2: the most
# rows that the solver with its matrices in registers takes
@pytest.mark.parametrize("side", [8, 16, 22, 23, 32, 45])
@pytest.mark.parametrize("dt", sorted(TYPES))
@pytest.mark.parametrize("device", [False, True])
def test_one_workgroup_stencil_solver(gpu_lib, side, dt, device):
    pcg = gpu_lib
    A, b = _indefinite(side), inputs.rhs(side * side, 5)
    got = _solve(pcg, A, b, device, **TYPES[dt])
    _check(A, b, got, _solve(pcg, A, b, device, wg_max_n=-1, **TYPES[dt]), dt == "f64")


# in CSR the solver that walks the matrices in memory: single systems up to 512
# rows, and systems of a batch on both sides of the vectors' LDS bound
@pytest.mark.parametrize("side", [8, 22, 23, 45])
@pytest.mark.parametrize("dt", sorted(TYPES))
def test_one_workgroup_solver(gpu_lib, side, dt):
    pcg = gpu_lib
    A, b = _indefinite(side), inputs.rhs(side * side, 5)
    kw = dict(layout="csr", **TYPES[dt])
    want = _solve(pcg, A, b, False, wg_max_n=-1, **kw)
    _check(A, b, _solve(pcg, A, b, False, wg_max_n=512, **kw), want, dt == "f64")
    _check(A, b, _batch(pcg, A, b, **kw), want, dt == "f64")
    _check(A, b, _batch(pcg, A, b, wg_max_n_batch=-1, **kw), want, dt == "f64")
