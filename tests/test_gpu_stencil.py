"""Iteration kernels over stencil storage: with the automatic layout a
matrix of a few diagonals is solved from one triangle of A and from G^T's
values alone. Every solve has to equal the general kernels' (the
sliced-diagonal layout asked for) bit for bit, at the edges of tiles and for
every number of diagonals, storage type and option."""
import numpy as np
import pytest

import oracle
from paper_2510_27517_amd import inputs
from paper_2510_27517_amd.inputs import CSR

pytestmark = pytest.mark.gpu


def _banded(n, offsets, seed, skew=0.0):
    """Diagonally dominant matrix with entries at the given distances;
    skew != 0 makes one upper entry differ from its lower counterpart."""
    import scipy.sparse as sp

    rng = np.random.default_rng(seed)
    m = sp.csr_matrix((n, n))
    for o in (o for o in offsets if o < n):
        v = -rng.uniform(0.05, 1.0, n - o)
        m = m + sp.diags([v, v], [o, -o], shape=(n, n))
    d = np.asarray(abs(m).sum(axis=1)).ravel() + rng.uniform(0.5, 1.5, n)
    m = (m + sp.diags([d], [0], shape=(n, n))).tocsr()
    m.sort_indices()
    if skew:
        i = n // 2
        k = m.indptr[i + 1] - 1
        m.data[k] *= 1.0 + skew
    return CSR.from_scipy(m)


def _both(pcg, A, kind=None, G=None, tol=1e-9, maxit=300, x0=None, eps=0.0, seed=5, **kw):
    """The solve with the automatic layout and with sliced diagonals."""
    b = inputs.rhs(A.n, seed)
    out = []
    for layout in ("auto", "sdia"):
        with pcg.Solver(pcg.default_config(layout=layout, wg_max_n=-1, eps=eps, **kw)) as s:
            s.set_matrix(A)
            if G is not None:
                s.set_precond(G)
            else:
                s.build_precond(pcg.G_FSAI if kind is None else kind)
            out.append(s.solve(b, x0, tol=tol, maxit=maxit, allow_failure=True))
    a, g = out
    assert (a.status, a.iters, a.restarts, a.outer_iters) == (g.status, g.iters, g.restarts, g.outer_iters)
    assert np.array_equal(a.x, g.x, equal_nan=True)
    assert a.relres_true == g.relres_true or (np.isnan(a.relres_true) and np.isnan(g.relres_true))
    return a, g, b


# one tile is 128 rows in FP64 and 256 in FP32; far diagonals make every tile
# touch an end of the matrix
@pytest.mark.parametrize("n", [2, 63, 127, 128, 129, 255, 256, 257, 511, 513, 1025, 5000, 40003])
@pytest.mark.parametrize("offsets", [(), (1,), (1, 9), (1, 9, 100), (2, 3, 50, 300)])
def test_sizes_and_diagonals_fp64(gpu_lib, n, offsets):
    pcg = gpu_lib
    A = _banded(n, offsets, n)
    a, g, b = _both(pcg, A)
    if n >= 5000 and offsets:  # the half of A and G^T for both products: fewer bytes, so it was this path
        assert a.bytes_per_iter < g.bytes_per_iter
    if n <= 5000:
        with pcg.Solver(pcg.default_config(wg_max_n=-1)) as s:
            s.set_matrix(A)
            G = oracle.fsai_g(A)
            s.set_precond(G)
            got = s.solve(b, tol=1e-9, maxit=300)
        ref = oracle.pcg(A, G, b, tol=1e-9, maxit=300, delta_form=1)
        assert got.iters == ref.iters and np.array_equal(got.x, ref.x)


@pytest.mark.parametrize("n", [2, 255, 257, 1023, 20011])
@pytest.mark.parametrize("types", [("f64", "f64", "f32"), ("f64", "f64", "bf16"), ("f64", "f64", "f16"),
                                   ("f32", "f32", "f32"), ("f32", "f32", "bf16"), ("f32", "f32", "f16")])
def test_storage_types(gpu_lib, n, types):
    pcg = gpu_lib
    v, a, g = types
    _both(pcg, _banded(n, (1, 2, 33), n), vec_dtype=v, a_dtype=a, g_dtype=g, tol=1e-5)
    if v == "f32":
        _both(pcg, _banded(n, (1, 2, 33), n), vec_dtype=v, a_dtype=a, g_dtype=g, refine=1, tol=1e-9)


@pytest.mark.parametrize("case", ["eps_rr", "odd_chunk", "plain_launches", "restart", "jacobi", "identity", "fixed",
                                  "maxit", "x0", "nan", "zero", "grid1", "cache_off", "device_fsai"])
def test_options(gpu_lib, case):
    pcg = gpu_lib
    A = inputs.poisson(3, 14, 1.0, 12)
    if case == "eps_rr":  # replacement through the general kernels between ordinary iterations
        _both(pcg, A, eps=0.05, rr_period=7)
    elif case == "odd_chunk":  # iteration parity differs from chunk to chunk
        _both(pcg, A, graph_iters=5, rr_period=25)
        _both(pcg, A, graph_iters=7, rr_period=0)
    elif case == "plain_launches":
        _both(pcg, A, graph_iters=0)
    elif case == "restart":
        # a system and right-hand side whose recurrence is known to drift (the oracle restarts once)
        a, _, _ = _both(pcg, inputs.poisson(3, 12, 2.5, 1), rr_period=0, tol=1e-13, maxit=5000, seed=11)
        assert a.restarts >= 1
    elif case in ("jacobi", "identity", "fixed"):
        _both(pcg, A, kind={"jacobi": pcg.G_JACOBI, "identity": pcg.G_IDENTITY, "fixed": pcg.G_FIXED}[case])
    elif case == "maxit":
        for m in (0, 1, 2, 11):
            _both(pcg, A, maxit=m)
    elif case == "x0":
        _both(pcg, A, x0=np.linspace(-1.0, 1.0, A.n))
    elif case in ("nan", "zero"):
        with pcg.Solver(pcg.default_config(wg_max_n=-1)) as s:
            s.set_matrix(A)
            s.build_precond(pcg.G_FSAI)
            b = np.zeros(A.n)
            if case == "nan":
                b[17] = np.nan
            got = s.solve(b, tol=1e-8, maxit=50, allow_failure=True)
            assert got.status == (pcg.EBREAKDOWN if case == "nan" else pcg.OK)
            again = s.solve(inputs.rhs(A.n, 1), tol=1e-8, maxit=500)  # the context still solves
            assert again.status == pcg.OK
    elif case == "grid1":
        _both(pcg, inputs.poisson(2, 90, 1.0, 3), grid_mult=1)
    elif case == "cache_off":
        _both(pcg, A, cache_mb=-1)
        _both(pcg, A, cache_mb=1)
    else:
        _both(pcg, A, g_device=1)


def test_what_the_stencil_storage_does_not_take(gpu_lib):
    """An A that is not symmetric bit for bit, a G with both triangles and a
    matrix of too many diagonals keep to the general kernels, and a context
    that changes between such systems and stencils solves each right."""
    pcg = gpu_lib
    n = 3000
    sym = _banded(n, (1, 9), 1)
    skew = _banded(n, (1, 9), 1, skew=1e-15)
    assert not np.array_equal(skew.val, sym.val)
    wide = _banded(n, (1, 2, 3, 4, 5, 6), 2)
    b = inputs.rhs(n, 5)
    want = {}
    for name, A in (("sym", sym), ("skew", skew), ("wide", wide)):
        a, g, _ = _both(pcg, A)
        want[name] = g.x
        if name == "skew":
            full = a.bytes_per_iter
        if name == "sym":
            half = a.bytes_per_iter
        if name == "wide":
            assert a.bytes_per_iter == g.bytes_per_iter
    assert half < full  # A's half is read only when A is symmetric
    # G = A's own pattern, both triangles
    G = CSR(sym.rowptr, sym.col, sym.val / 4.0)
    a, g, _ = _both(pcg, sym, G=G, maxit=40)
    with pcg.Solver(pcg.default_config(wg_max_n=-1)) as s:
        for name, A in (("sym", sym), ("wide", wide), ("skew", skew), ("sym", sym)):
            s.set_matrix(A)
            s.build_precond(pcg.G_FSAI)
            assert np.array_equal(s.solve(b, tol=1e-9, maxit=300).x, want[name])
        s.set_precond(G)  # the same A, another G: the general G kernels after the stencil ones
        assert np.array_equal(s.solve(b, tol=1e-9, maxit=40).x, g.x)
        s.build_precond(pcg.G_FSAI)
        assert np.array_equal(s.solve(b, tol=1e-9, maxit=300).x, want["sym"])
