"""The losses over every kind of launch: lane groups of each size, one and two
probes per lane on either side of the wave count that decides, batches of
four, three and two entries with each remainder, and launches of less than one
turn of rows per wave. Compared with the same sums in NumPy."""
import numpy as np
import pytest

from paper_2510_27517_amd import inputs
from paper_2510_27517_amd.inputs import CSR

pytestmark = pytest.mark.gpu


def _random(n, per_row, seed):
    import scipy.sparse as sp

    rng = np.random.default_rng(seed)
    m = n * per_row // 2
    A = sp.coo_matrix((rng.uniform(-1.0, 0.0, m), (rng.integers(0, n, m), rng.integers(0, n, m))), (n, n)).tocsr()
    A = A + A.T
    A.setdiag(0.0)
    A.eliminate_zeros()
    A = (A + sp.diags(-np.asarray(A.sum(axis=1)).ravel() * 1.05 + 0.1)).tocsr()
    A.sort_indices()
    return CSR.from_scipy(A)


SYSTEMS = {
    "one_row": lambda: _random(1, 0, 1),
    "csr_70": lambda: _random(70, 9, 2),
    "csr_3000": lambda: _random(3000, 40, 3),
    "elasticity_7": lambda: inputs.elasticity(7, seed=4),
    "elasticity_27": lambda: inputs.elasticity(27, seed=5),
    "grid_2d": lambda: inputs.poisson(2, 61, 1.0, 6),
    "grid_3d": lambda: inputs.poisson(3, 41, 1.0, 7),
}
_cache = {}


def _system(name):
    if name not in _cache:
        A = SYSTEMS[name]()
        # G on tril(A) as the library's fixed kind: entries of A's size, any sign
        import scipy.sparse as sp

        M = A.to_scipy()
        L = sp.tril(M, format="csr")
        d = 1.0 / np.sqrt(M.diagonal())
        G = CSR.from_scipy((sp.diags(d) @ L @ sp.diags(d)).T.tocsr())
        _cache[name] = (A, G)
    return _cache[name]


# 65,536 rows hold 4,096 waves of groups of four; 59,049 and 68,921 rows lie on
# either side of it at 8 probes
@pytest.mark.parametrize("name,layout", [(n, "auto") for n in sorted(SYSTEMS)] + [
    (n, l) for n in ("one_row", "csr_70", "csr_3000", "elasticity_7", "grid_2d") for l in ("csr", "sell")])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 6, 8, 9, 16, 17, 32, 33, 64, 100])
def test_losses(gpu_lib, name, layout, k):
    import torch

    pcg = gpu_lib
    A, G = _system(name)
    eps = 0.01
    W = np.random.default_rng(k).standard_normal((A.n, k))
    M, g = A.to_scipy(), G.to_scipy()
    U = g @ (g.T @ W) + eps * W
    Y = M @ U
    na = np.abs(A.val[A.val != 0]).mean()
    want = {"sai": ((Y / na - W) ** 2).sum(0), "l2": ((Y - W) ** 2).sum(0),
            "cs": (W * Y).sum(0) / np.sqrt((W * W).sum(0) * (Y * Y).sum(0))}
    with pcg.Solver(pcg.default_config(layout=layout, eps=eps)) as s:
        s.set_matrix(A)
        s.set_precond(G)
        Wd = torch.from_numpy(W).cuda()
        got, host = s.sai_loss(Wd), s.sai_loss(W)
        small = s.sai_loss_noalloc(Wd) if A.n * k < 2_000_000 else got
    # three products and a sum in FP64: n u^(1/2)-like growth stays far below 1e-11
    for q in want:
        scale = np.abs(want[q]) if q != "cs" else np.maximum(np.abs(want[q]), 1e-2)
        assert (np.abs(got[q] - want[q]) <= 1e-11 * scale).all(), (q, got[q], want[q])
        assert np.array_equal(got[q], host[q]) and np.array_equal(got[q], small[q])
