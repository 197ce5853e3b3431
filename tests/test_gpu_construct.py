"""Construction: FSAI on the device with one thread per short row, and the
host's layouts made by several threads, against the host builder and the
oracle."""
import numpy as np
import pytest

import oracle
from paper_2510_27517_amd import inputs
from paper_2510_27517_amd.inputs import CSR
from test_gpu_stencil import _banded

pytestmark = pytest.mark.gpu


def _products(pcg, A, x, **kw):
    out = []
    for dev in (1, 0):
        with pcg.Solver(pcg.default_config(g_device=dev, **kw)) as s:
            s.set_matrix(A)
            s.build_precond(pcg.G_FSAI)
            out.append([s.matvec(op, x) for op in (pcg.OP_A, pcg.OP_GT, pcg.OP_G)])
    return out


# tril rows of up to 1 .. 10 entries: one thread per row up to 8, a wave above
@pytest.mark.parametrize("reach", [0, 1, 2, 3, 6, 7, 8, 9])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 1000, 5003])
def test_device_fsai_row_lengths(gpu_lib, n, reach):
    pcg = gpu_lib
    A = _banded(n, tuple(range(1, reach + 1)), n + reach)
    x = np.random.default_rng(1).standard_normal(n)
    for layout in ("auto", "csr"):
        dev, host = _products(pcg, A, x, layout=layout)
        for d, h in zip(dev, host):
            assert np.array_equal(d, h)


def test_device_fsai_reports_a_pivot_that_is_not_positive(gpu_lib):
    pcg = gpu_lib
    A = _banded(500, (1, 9), 2)
    A.val[A.rowptr[77]:A.rowptr[78]] *= -1.0
    with pcg.Solver(pcg.default_config(g_device=1)) as s:
        s.set_matrix(A)
        with pytest.raises(pcg.PCGError) as e:
            s.build_precond(pcg.G_FSAI)
        assert e.value.status == pcg.EBREAKDOWN


# from 32,768 rows the layouts are made by several threads, each its slices
@pytest.mark.parametrize("n", [32767, 32768, 49217, 100003])
@pytest.mark.parametrize("case", ["stencil", "mixed_f16", "graph"])
def test_layouts_made_by_threads(gpu_lib, n, case):
    pcg = gpu_lib
    A = inputs.rgg_laplacian(n, 3) if case == "graph" else _banded(n, (1, 5, 77), n)
    x = np.random.default_rng(1).standard_normal(n)
    G = oracle.fsai_g(A)
    kw = dict(vec_dtype="f32", a_dtype="f32", g_dtype="f16") if case == "mixed_f16" else {}
    with pcg.Solver(pcg.default_config(**kw)) as s:
        s.set_matrix(A)
        s.set_precond(G)
        got = [s.matvec(op, x) for op in (pcg.OP_A, pcg.OP_GT, pcg.OP_G)]
    if case == "mixed_f16":
        with pcg.Solver(pcg.default_config(layout="csr", **kw)) as s:
            s.set_matrix(A)
            s.set_precond(G)
            want = [s.matvec(op, x) for op in (pcg.OP_A, pcg.OP_GT, pcg.OP_G)]
    else:
        want = [oracle.spmv(A, x), oracle.spmv_t(G, x), oracle.spmv(G, x)]
    for a, b in zip(got, want):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("what", ["column", "order", "diagonal", "rowptr", "count"])
def test_a_large_malformed_matrix_is_refused_as_before(gpu_lib, what):
    pcg = gpu_lib
    A = _banded(60000, (1, 5), 1)
    rp, ci, v = A.rowptr.copy(), A.col.copy(), A.val.copy()
    at = int(rp[51234])
    if what == "column":
        ci[at] = 60000
        text = f"column out of range (at {at})"
    elif what == "order":
        ci[at + 1] = ci[at]
        text = f"columns not strictly ascending (at {at + 1})"
    elif what == "diagonal":
        k = at + int(np.flatnonzero(ci[at:rp[51235]] == 51234)[0])
        ci, v = np.delete(ci, k), np.delete(v, k)
        rp[51235:] -= 1
        text = "missing diagonal entry (at 51234)"
    elif what == "rowptr":
        rp[51234] = rp[51236] + 1  # row 51233 then runs into the next rows' columns, which comes first
        text = "columns not strictly ascending"
    else:
        rp[-1] -= 1
        text = "rowptr[n] != nnz"
    with pcg.Solver() as s:
        with pytest.raises(pcg.PCGError) as e:
            s.set_matrix(rowptr=rp, col=ci, val=v)
        assert e.value.status == pcg.EINVAL and text in str(e.value), str(e.value)
        s.set_matrix(CSR(A.rowptr, A.col, A.val))
        s.build_precond(pcg.G_FSAI)
        assert s.solve(inputs.rhs(A.n, 1), tol=1e-8, maxit=500).status == pcg.OK
