"""pcg_time_kernels runs on the last solve's right-hand side, whichever
solver that solve took and wherever its vectors were."""
import numpy as np
import pytest

from paper_2510_27517_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side", [8, 45, 46])  # one wave; the largest and one too large for one workgroup
@pytest.mark.parametrize("types", [{}, dict(vec_dtype="f32", a_dtype="f32", g_dtype="f16")], ids=["f64", "f32"])
def test_device_solve_is_the_last(gpu_lib, side, types):
    import torch

    pcg = gpu_lib
    A = inputs.poisson(2, side, 1.0, 7)
    b = inputs.rhs(A.n, 5)
    with pcg.Solver(pcg.default_config(**types)) as s:
        s.set_matrix(A)
        s.build_precond(pcg.G_FSAI)
        s.solve(np.zeros(A.n), tol=1e-4, maxit=300)
        s.solve(torch.from_numpy(b).cuda(), tol=1e-4, maxit=300)
        assert min(s.time_kernels(3)["ms"]) > 0.0
        s.solve(torch.zeros(A.n, dtype=torch.float64, device="cuda"), tol=1e-4, maxit=300)
        with pytest.raises(pcg.PCGError) as e:
            s.time_kernels(3)
        assert e.value.status == pcg.ESTATE
