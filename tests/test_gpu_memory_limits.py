"""The stencil storage of a single system is a second copy of its values: it
never keeps from the caller what fits without it. Each piece of work runs
once with sliced diagonals asked for (no stencil storage), then with the
automatic layout in exactly the device memory that the first run needed."""
import numpy as np
import pytest

from paper_2510_27517_amd import inputs
from paper_2510_27517_amd.inputs import CSR

pytestmark = pytest.mark.gpu


def _allocator(pcg, limit=None):
    class Limited(pcg.TorchAllocator):
        """Counts the bytes held; refuses what would pass the limit."""

        def __init__(self):
            super().__init__(0)
            self.peak = self.refused = 0
            inner = self.alloc_fn

            def alloc(nbytes, user):
                held = sum(self.live.values()) + int(nbytes)
                if limit is not None and held > limit:
                    self.refused += 1
                    return None
                self.peak = max(self.peak, held)
                return inner(nbytes, user)

            self.alloc_fn = pcg.ALLOC_FN(alloc)

    return Limited()


def _work(pcg, what, s, A, b):
    """The results of the work and a solve before and after it."""
    if what == "escalation":
        r = s.solve(b, tol=1e-6, maxit=20000)
        assert r.escalated == 1
        return [r.x, s.solve(b, tol=1e-6, maxit=20000).x]
    out = [s.solve(b, tol=1e-8, maxit=500).x]
    if what == "loss":
        out += list(s.sai_loss(np.random.default_rng(1).standard_normal((A.n, 5))).values())
    elif what == "precond":
        s.build_precond(pcg.G_SEEDED, 3)
        out.append(s.matvec(pcg.OP_MINV, b))
        s.build_precond(pcg.G_FSAI)
    elif what == "batch":
        # one system: how many are admitted together, each with scratch of its
        # own, depends on when their preparation ends
        out += [x for x, _ in s.solve_batch([dict(A=A, b=b, tol=1e-8, maxit=500)])]
    out.append(s.solve(b, tol=1e-8, maxit=500).x)
    return out


def _near_singular(side):
    """A grid's Laplacian without boundary, shifted a little: FP32 inner solves
    fail on it, so refinement goes on with FP64 ones in vectors of their own."""
    import scipy.sparse as sp

    one = sp.diags([-np.ones(side - 1), -np.ones(side - 1)], [-1, 1])
    W = sp.kron(one, sp.identity(side)) + sp.kron(sp.identity(side), one)
    M = (W + sp.diags(-np.asarray(W.sum(axis=1)).ravel() + 1e-7)).tocsr()
    M.sort_indices()
    return CSR.from_scipy(M)


@pytest.mark.parametrize("what", ["loss", "precond", "batch", "escalation"])
@pytest.mark.parametrize("g_device", [0, 1])
def test_runs_in_the_memory_it_needed(gpu_lib, what, g_device):
    pcg = gpu_lib
    A = inputs.poisson(2, 120, 1.0, 3) if what != "escalation" else _near_singular(120)
    b = inputs.rhs(A.n, 4)
    types = dict(vec_dtype="f32", a_dtype="f32", g_dtype="bf16", refine=1) if what == "escalation" else {}

    def run(layout, limit):
        al = _allocator(pcg, limit)
        with pcg.Solver(pcg.default_config(layout=layout, g_device=g_device, mem_budget_mb=16, **types),
                        allocator=al) as s:
            s.set_matrix(A)
            s.build_precond(pcg.G_FSAI)
            return _work(pcg, what, s, A, b), al

    want, first = run("sdia", None)
    got, second = run("auto", first.peak)
    assert second.peak <= first.peak
    assert len(got) == len(want) and all(np.array_equal(g, w) for g, w in zip(got, want))
    assert not first.live and not second.live
