"""One-workgroup solver with the matrices in registers (small systems of few
diagonals): every solve equals the three-kernel iteration's bit for bit, at
the edges of its workgroup sizes and for each type and option."""
import numpy as np
import pytest

import oracle
from paper_2510_27517_amd import inputs
from test_gpu_stencil import _banded

pytestmark = pytest.mark.gpu


def _pair(pcg, A, tol=1e-9, maxit=300, x0=None, seed=5, device=False, kind=None, **kw):
    b = inputs.rhs(A.n, seed)
    out = []
    for wg in (512, -1):
        with pcg.Solver(pcg.default_config(wg_max_n=wg, layout=kw.pop("layout", "sdia"), **kw)) as s:
            s.set_matrix(A)
            s.build_precond(pcg.G_FSAI if kind is None else kind)
            if device:
                import torch

                x0d = None if x0 is None else torch.from_numpy(x0).cuda()
                r = s.solve(torch.from_numpy(b).cuda(), x0d, tol=tol, maxit=maxit, allow_failure=True)
                r.x = r.x.cpu().numpy()
            else:
                r = s.solve(b, x0, tol=tol, maxit=maxit, allow_failure=True)
            out.append(r)
    a, g = out
    assert (a.status, a.iters, a.restarts, a.outer_iters, a.escalated) == \
        (g.status, g.iters, g.restarts, g.outer_iters, g.escalated)
    assert np.array_equal(a.x, g.x, equal_nan=True)
    if a.status >= 0:
        assert a.relres_true == g.relres_true and a.relres_rec == g.relres_rec
    return a, b


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049])
@pytest.mark.parametrize("offsets", [(), (1,), (1, 9), (1, 9, 100)])
def test_sizes(gpu_lib, n, offsets):
    pcg = gpu_lib
    A = _banded(n, offsets, n)
    a, b = _pair(pcg, A, device=bool(n % 2))
    _pair(pcg, A, tol=1e-5, vec_dtype="f32", a_dtype="f32", g_dtype="bf16", device=bool(n % 2))
    with pcg.Solver(pcg.default_config(layout="sdia")) as s:
        s.set_matrix(A)
        G = oracle.fsai_g(A)
        s.set_precond(G)
        got = s.solve(b, tol=1e-9, maxit=300)
    ref = oracle.pcg(A, G, b, tol=1e-9, maxit=300, delta_form=1)
    assert got.iters == ref.iters and np.array_equal(got.x, ref.x)


@pytest.mark.parametrize("side", [20, 45])
@pytest.mark.parametrize("case", ["eps_rr", "restart", "maxit", "x0", "nan", "zero", "not_spd", "jacobi", "f32", "f16",
                                  "f64_bf16", "refined", "same_buffer"])
def test_options(gpu_lib, side, case):
    pcg = gpu_lib
    A = inputs.poisson(2, side, 1.0, 7)
    rng = np.random.default_rng(3)
    if case == "eps_rr":
        _pair(pcg, A, eps=0.05, rr_period=7, device=True)
    elif case == "restart":  # the case known to restart from its true residual once
        a, _ = _pair(pcg, inputs.poisson(3, 8, 2.5, 1), tol=1e-14, maxit=5000, rr_period=0, seed=11)
        b, _ = _pair(pcg, inputs.poisson(2, side, 2.5, 1), tol=1e-14, maxit=3000, rr_period=0, seed=11)
        assert a.restarts + b.restarts >= 1
    elif case == "maxit":
        for m in (0, 1, 5):
            _pair(pcg, A, maxit=m, device=True)
    elif case == "x0":
        _pair(pcg, A, x0=rng.standard_normal(A.n))
        _pair(pcg, A, x0=rng.standard_normal(A.n), device=True)
    elif case in ("nan", "zero", "same_buffer"):
        import torch

        with pcg.Solver(pcg.default_config()) as s:
            s.set_matrix(A)
            s.build_precond(pcg.G_FSAI)
            b = np.zeros(A.n)
            if case == "nan":
                b[3] = np.nan
            if case != "same_buffer":
                r = s.solve(torch.from_numpy(b).cuda(), torch.ones(A.n, device="cuda"), tol=1e-8, maxit=50,
                            allow_failure=True)
                assert r.status == (pcg.EBREAKDOWN if case == "nan" else pcg.OK)
                if case == "zero":
                    assert not r.x.cpu().numpy().any()
            b = inputs.rhs(A.n, 1)
            want = s.solve(b, b, tol=1e-8, maxit=500).x
            bx = torch.from_numpy(b).cuda()  # the right-hand side's own buffer as x0 and solution
            import ctypes

            res = pcg.Result()
            st = s._lib.pcg_solve(s._h, bx.data_ptr(), bx.data_ptr(), 1e-8, 500, 1, ctypes.byref(res))
            assert st == pcg.OK and np.array_equal(bx.cpu().numpy(), want)
    elif case == "not_spd":
        B = _banded(side * side, (1, 9), 1)
        B.val[B.rowptr[4]:B.rowptr[5]] *= -1.0
        a, _ = _pair(pcg, B, kind=pcg.G_IDENTITY, device=True)
        assert a.status == pcg.EBREAKDOWN
    elif case == "jacobi":
        _pair(pcg, A, kind=pcg.G_JACOBI)
    elif case in ("f32", "f16"):
        _pair(pcg, A, tol=1e-4, vec_dtype="f32", a_dtype="f32", g_dtype=case, device=True)
    elif case == "f64_bf16":
        _pair(pcg, A, g_dtype="bf16", device=True)
    else:
        _pair(pcg, A, tol=1e-11, vec_dtype="f32", a_dtype="f32", g_dtype="bf16", refine=1, device=True)
