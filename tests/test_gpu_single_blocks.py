"""The single system's kernels built for 3x3 blocks give the batch's kernels'
solution (built for every layout) and, in FP64, the oracle's, bit for bit:
slices of 21 block rows that end unevenly, and one block alone."""
import functools

import numpy as np
import pytest

import oracle
from paper_2510_27517_amd import inputs
from paper_2510_27517_amd.inputs import CSR

pytestmark = pytest.mark.gpu


def _blocked(nb, per_row, seed):
    """Diagonally dominant, `nb` block rows of about `per_row` full 3x3 blocks."""
    import scipy.sparse as sp

    rng = np.random.default_rng(seed)
    m = nb * per_row // 2
    W = sp.coo_matrix((np.ones(m), (rng.integers(0, nb, m), rng.integers(0, nb, m))), (nb, nb)).tocsr()
    W = ((W + W.T + sp.identity(nb)) > 0).astype(float)
    M = sp.kron(W, np.ones((3, 3))).tocsr()
    M.data = -rng.uniform(0.1, 1.0, M.nnz)
    M = (M + M.T).tocsr()
    M = (M + sp.diags(np.asarray(abs(M).sum(axis=1)).ravel() * 2.0)).tocsr()
    M.sort_indices()
    return CSR.from_scipy(M)


@functools.lru_cache(maxsize=None)
def _system(name):
    A = inputs.elasticity(name, seed=name) if isinstance(name, int) else _blocked(*name)
    return A, oracle.fsai_g(A)


@pytest.mark.parametrize("name", [(1, 0, 1), (20, 3, 2), (21, 3, 3), (22, 3, 4), (1500, 9, 5), 3, 6])
@pytest.mark.parametrize("types", [{}, dict(vec_dtype="f32", a_dtype="f32", g_dtype="bf16"),
                                   dict(vec_dtype="f32", a_dtype="f32", g_dtype="f32")],
                         ids=["f64", "f32-bf16", "f32"])
@pytest.mark.parametrize("uw", [4, 8])
def test_single_equals_batch_and_oracle(gpu_lib, name, types, uw):
    pcg = gpu_lib
    A, G = _system(name)
    b = inputs.rhs(A.n, 3)
    kw = dict(layout="bsr3", wg_max_n=-1, wg_max_n_batch=-1, loads_in_flight=uw, eps=0.01, **types)
    tol = 1e-4 if types else 1e-9
    with pcg.Solver(pcg.default_config(**kw)) as s:
        s.set_matrix(A)
        s.set_precond(G)
        one = s.solve(b, tol=tol, maxit=200)
    with pcg.Solver(pcg.default_config(mem_budget_mb=64, **kw)) as s:
        many = s.solve_batch([dict(A=A, G=G, b=b, tol=tol, maxit=200)] * 2)
    for x, r in many:
        assert r["iters"] == one.iters and np.array_equal(x, one.x)
    if not types:
        ref = oracle.pcg(A, G, b, eps=0.01, tol=tol, maxit=200, delta_form=1)
        assert one.iters == ref.iters and np.array_equal(one.x, ref.x)
