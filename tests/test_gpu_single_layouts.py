"""A single system's iteration kernels are built for one layout each: every
layout, storage type and loads-in-flight setting has to give the batch's
kernels' solution (built for all layouts) and, in FP64, the oracle's, bit for
bit, where blocks and slices end unevenly."""
import functools

import numpy as np
import pytest

import oracle
from paper_2510_27517_amd import inputs
from paper_2510_27517_amd.inputs import CSR

pytestmark = pytest.mark.gpu


def _matrix(n, degree, long_row, seed):
    """Diagonally dominant, about `degree` random entries per row; one row
    (and column) of `long_row` entries."""
    import scipy.sparse as sp

    rng = np.random.default_rng(seed)
    nnz = n * degree // 2
    m = sp.coo_matrix((rng.uniform(0.1, 1.0, nnz), (rng.integers(0, n, nnz), rng.integers(0, n, nnz))), (n, n)).tocsr()
    if long_row:
        j = np.sort(rng.choice(n, long_row, replace=False))
        m = m + sp.coo_matrix((rng.uniform(0.1, 1.0, j.size), (np.full(j.size, n // 2), j)), (n, n)).tocsr()
    m = -(m + m.T)
    m.setdiag(0.0)
    m.eliminate_zeros()
    m = (m + sp.diags(np.asarray(abs(m).sum(axis=1)).ravel() + rng.uniform(0.5, 1.5, n))).tocsr()
    m.sort_indices()
    return CSR.from_scipy(m)


@functools.lru_cache(maxsize=None)
def _system(n, degree, long_row):
    A = _matrix(n, degree, long_row, n)
    return A, oracle.fsai_g(A)


# one slice is 64 rows; a row block holds at most 256 rows and 2048 products in
# FP64 (4096 in FP32), staged in rounds of 2048: rows alone end a block (degree
# 2), products do (degree 30), a row exceeds a block; A's CSR rows too long for
# the kernels of one layout, but not G's (degree 300)
@pytest.mark.parametrize("layout", ["csr", "sell"])
@pytest.mark.parametrize("uw", [4, 8])
@pytest.mark.parametrize("types", [{}, dict(vec_dtype="f32", a_dtype="f32", g_dtype="bf16"),
                                   dict(vec_dtype="f32", a_dtype="f32", g_dtype="f32")],
                         ids=["f64", "f32-bf16", "f32"])
@pytest.mark.parametrize("n,degree,long_row", [(1, 0, 0), (65, 4, 0), (257, 2, 0), (1000, 30, 0), (5003, 13, 4500),
                                               (1200, 300, 0)])
def test_single_equals_batch_and_oracle(gpu_lib, layout, uw, types, n, degree, long_row):
    pcg = gpu_lib
    A, G = _system(n, degree, long_row)
    b = inputs.rhs(A.n, 3)
    kw = dict(layout=layout, wg_max_n=-1, wg_max_n_batch=-1, loads_in_flight=uw, eps=0.01, **types)
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
