"""Products outside the iteration: pcg_matvec on device vectors in place and
through staging, and the losses' multi-probe products at the edges of their
lane groups and probe chunks."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_2510_27517_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("types", [("f64", "f64", "f64"), ("f64", "f64", "f16"), ("f32", "f32", "f32"),
                                   ("f32", "f32", "bf16"), ("f32", "f32", "f16")])
@pytest.mark.parametrize("layout", ["auto", "csr", "sell"])
def test_matvec_device_host_and_overlap(gpu_lib, types, layout):
    """A device product equals the host one (staged) bit for bit, with y apart
    from x, the same as x, and half over it; M^-1 x is its two products."""
    import torch

    pcg = gpu_lib
    v, a, g = types
    A = inputs.rgg_laplacian(3001, 3) if layout != "auto" else inputs.elasticity(6, 1.0, 0.3, 2)
    x = np.random.default_rng(2).standard_normal(A.n)
    with pcg.Solver(pcg.default_config(layout=layout, vec_dtype=v, a_dtype=a, g_dtype=g, eps=0.125)) as s:
        s.set_matrix(A)
        s.build_precond(pcg.G_FSAI)
        for op in (pcg.OP_A, pcg.OP_GT, pcg.OP_G, pcg.OP_MINV):
            want = s.matvec(op, x)
            xd = torch.from_numpy(x).cuda()
            assert np.array_equal(s.matvec(op, xd).cpu().numpy(), want)
            assert np.array_equal(xd.cpu().numpy(), x)
            for shift in (0, A.n // 2, 1):
                buf = torch.zeros(2 * A.n, dtype=torch.float64, device="cuda")
                buf[:A.n] = xd
                torch.cuda.synchronize()
                st = s._lib.pcg_matvec(s._h, op, ctypes.c_void_p(buf.data_ptr()),
                                       ctypes.c_void_p(buf.data_ptr() + 8 * shift), 1)
                assert st == pcg.OK
                assert np.array_equal(buf[shift:shift + A.n].cpu().numpy(), want), (op, shift)
        if types == ("f64", "f64", "f64"):
            t = s.matvec(pcg.OP_G, s.matvec(pcg.OP_GT, x))
            assert np.array_equal(s.matvec(pcg.OP_MINV, x), 1.0 * t + 0.125 * x)


def test_matvec_leaves_what_rows_do_not_read_alone(gpu_lib):
    """A NaN or infinity in x reaches the rows that read it, and no row of
    another slice."""
    pcg = gpu_lib
    A = inputs.poisson(2, 40, 1.0, 3)
    x = np.ones(A.n)
    x[700] = np.inf
    x[900] = np.nan
    with pcg.Solver(pcg.default_config(layout="csr")) as s:
        s.set_matrix(A)
        s.build_precond(pcg.G_FSAI)
        y = s.matvec(pcg.OP_A, x)
    assert np.array_equal(y, oracle.spmv(A, x), equal_nan=True)


def _check(got, ref):
    for key in ("sai", "l2"):
        assert np.allclose(got[key], ref[key], rtol=1e-12, atol=0), key
    assert np.allclose(got["cs"], ref["cs"], rtol=0, atol=1e-12)


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 8, 9, 16, 17, 32, 33, 64, 65, 128, 130])
@pytest.mark.parametrize("case", ["sdia", "sell", "csr", "blocks"])
def test_loss_probe_counts(gpu_lib, k, case):
    import torch

    pcg = gpu_lib
    A = inputs.elasticity(5, 1.0, 0.3, 4) if case == "blocks" else inputs.poisson(3, 11, 1.0, 4)
    W = inputs.normal(k, inputs.STREAM_PROBE, A.n * k).reshape(A.n, k)
    with pcg.Solver(pcg.default_config(layout="bsr3" if case == "blocks" else case, eps=0.01)) as s:
        s.set_matrix(A)
        s.build_precond(pcg.G_FSAI)
        got = s.sai_loss(W)
        dev = s.sai_loss(torch.from_numpy(W).cuda())
    for key in got:
        assert np.array_equal(got[key], dev[key]), key
    _check(got, oracle.sai_losses(A, oracle.fsai_g(A), W, 0.01))


@pytest.mark.parametrize("n,k", [(68921, 66), (68921, 83), (9261, 450)])
def test_loss_in_chunks(gpu_lib, n, k):
    """Blocks large enough to go in chunks of probes, even and odd ones."""
    import torch

    pcg = gpu_lib
    A = inputs.poisson(3, round(n ** (1 / 3)), 1.0, 4)
    assert A.n == n
    W = inputs.normal(k, inputs.STREAM_PROBE, A.n * k).reshape(A.n, k)
    with pcg.Solver(pcg.default_config()) as s:
        s.set_matrix(A)
        s.build_precond(pcg.G_FSAI)
        got = s.sai_loss(torch.from_numpy(W).cuda())
    _check(got, oracle.sai_losses(A, oracle.fsai_g(A), W))
