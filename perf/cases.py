"""Performance cases of the FSAI-preconditioned CG library, through its public
Python binding (paper_2510_27517_amd.pcg).

Five kinds of work, the ones a program that uses the library has it do:
  solve      one linear system solved to a tolerance, A and the preconditioner
             already set, b and x on the GPU;
  batch      many independent systems from host memory solved together,
             preconditioners built by the library;
  apply      one product with A, G, G^T or the preconditioner M^-1 = G G^T,
             as inside a caller's own Krylov method;
  loss       the preconditioner-quality losses over Gaussian probes;
  construct  a new matrix set and its FSAI built, then applied once.
The systems are those of the benchmark and the tests: 2D and 3D lognormal
Poisson on grids, random-geometric-graph Laplacians, Q1 elasticity with three
unknowns per node, and the synthetic P P^T systems.
"""
import math

import numpy as np
import torch

from paper_2510_27517_amd import inputs, pcg

DEVICE = "cuda:0"
# device memory of a batch's pool: the largest batch here takes under 2 GB
POOL_MB = 4096

# storage types and refinement of a context: plain FP64, plain FP32, and FP32
# with a 16-bit G inside FP64 refinement
TYPES = {
    "f64": dict(vec_dtype="f64", a_dtype="f64", g_dtype="f64"),
    "f64_bf16": dict(vec_dtype="f64", a_dtype="f64", g_dtype="bf16"),
    "f32": dict(vec_dtype="f32", a_dtype="f32", g_dtype="f32"),
    "mixed_f32": dict(vec_dtype="f32", a_dtype="f32", g_dtype="f32", refine=1),
    "mixed_bf16": dict(vec_dtype="f32", a_dtype="f32", g_dtype="bf16", refine=1),
    "mixed_f16": dict(vec_dtype="f32", a_dtype="f32", g_dtype="f16", refine=1),
}
KINDS = {"fsai": pcg.G_FSAI, "block_fsai": pcg.G_BFSAI, "fixed": pcg.G_FIXED, "jacobi": pcg.G_JACOBI}
OPS = {"A": pcg.OP_A, "GT": pcg.OP_GT, "G": pcg.OP_G, "MINV": pcg.OP_MINV}
VALUE_BYTES = {"f64": 8, "f32": 4, "bf16": 2, "f16": 2}


def listed():
    return [
        # the smallest solves: a coarse grid or a subdomain problem, where the
        # call's latency is all that counts
        dict(name="solve_2d_8", do="solve", system="poisson2d", size=8, types="f64", precond="fsai", tol=1e-8),
        # small systems, called many times over by time steppers
        dict(name="solve_2d_45", do="solve", system="poisson2d", size=45, types="f64", precond="fsai", tol=1e-8),
        # the size of the paper's own systems (about 32k unknowns)
        dict(name="solve_2d_181", do="solve", system="poisson2d", size=181, types="f64", precond="fsai", tol=1e-8),
        # the headline workload
        dict(name="solve_3d_128", do="solve", system="poisson3d", size=128, types="f64", precond="fsai", tol=1e-8),
        # an ordinary 3D grid of odd side, mixed precision
        dict(name="solve_3d_101_mixed", do="solve", system="poisson3d", size=101, types="mixed_bf16", precond="fsai",
             tol=1e-8),
        # a structural-mechanics system, 3x3 blocks, 81 entries per row
        dict(name="solve_elasticity_40", do="solve", system="elasticity", size=40, types="f64", precond="fsai",
             tol=1e-8),
        # an irregular graph system, as the serving workload's requests
        dict(name="solve_rgg_150k", do="solve", system="rgg", size=150001, types="mixed_bf16", precond="fsai",
             tol=1e-6),
        # the paper's algebraic set: ragged rows, many iterations
        dict(name="solve_ppt_18000", do="solve", system="ppt", size=18000, types="f64", precond="fsai", tol=1e-8),
        # uneven 2D and 3D systems from host memory, solved together
        dict(name="batch_48", do="batch", count=48, max2d=256, max3d=64, types="mixed_f32", precond="fsai", tol=1e-6),
        # the preconditioner applied inside a caller's own method
        dict(name="apply_minv_3d_100", do="apply", system="poisson3d", size=100, types="f64", precond="fsai",
             op="MINV"),
        # the losses that score a preconditioner, at the benchmark's probe count
        dict(name="loss_3d_96_k32", do="loss", system="poisson3d", size=96, types="f64", precond="fsai", probes=32),
        # a new matrix: layouts, FSAI on the device and a first application
        dict(name="construct_3d_64", do="construct", system="poisson3d", size=64, types="f64", precond="fsai"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_system(rng, big):
    """A system name and size; big scales the largest sizes down."""
    system = rng.choice(["poisson2d", "poisson2d", "poisson3d", "poisson3d", "elasticity", "rgg"])
    lo, hi = {"poisson2d": (6, 700), "poisson3d": (4, 120), "elasticity": (3, 36), "rgg": (500, 300000)}[system]
    hi = int(hi * big) if system != "rgg" else int(hi * big * big * big)
    return system, _log_int(rng, lo, max(hi, lo + 1))


def draw(rng):
    do = rng.choice(["solve"] * 5 + ["apply", "apply", "loss", "batch", "construct"])
    if do == "batch":
        return dict(do=do, count=rng.randint(3, 40), max2d=_log_int(rng, 24, 256), max3d=_log_int(rng, 10, 64),
                    types=rng.choice(["mixed_f32", "mixed_bf16", "f64"]), precond="fsai", tol=1e-6)
    if do == "solve" and rng.random() < 0.12:
        return dict(do=do, system="ppt", size=_log_int(rng, 3000, 17000), types="f64", precond="fsai", tol=1e-8)
    system, size = _draw_system(rng, {"solve": 1.0, "apply": 1.0, "loss": 0.8, "construct": 0.55}[do])
    precond = "fsai"
    if do in ("solve", "apply") and rng.random() < 0.25:
        precond = rng.choice(["block_fsai", "jacobi"] if system == "elasticity" else ["fixed", "jacobi"])
    if do == "solve":
        types = rng.choice(["f64", "f64", "f64_bf16", "f32", "mixed_f32", "mixed_bf16", "mixed_f16"])
        # plain FP32 reaches 1e-5 only on well-conditioned, smaller systems
        if types == "f32" and size > {"poisson2d": 100, "poisson3d": 60, "elasticity": 12, "rgg": 20000}[system]:
            types = "mixed_f32"
        tol = 1e-5 if types == "f32" else rng.choice([1e-6, 1e-8])
        return dict(do=do, system=system, size=size, types=types, precond=precond, tol=tol)
    types = rng.choice(["f64", "f64", "f32"])
    if do == "apply":
        return dict(do=do, system=system, size=size, types=types, precond=precond,
                    op=rng.choice(["A", "GT", "G", "MINV", "MINV"]))
    if do == "loss":
        return dict(do=do, system=system, size=size, types=types, precond=precond, probes=_log_int(rng, 1, 48))
    return dict(do=do, system=system, size=size, types=types, precond=precond)


def _matrix(system, size, seed):
    if system == "poisson2d":
        return inputs.poisson(2, size, 1.0, seed)
    if system == "poisson3d":
        return inputs.poisson(3, size, 1.0, seed)
    if system == "elasticity":
        return inputs.elasticity(size, seed=seed)
    if system == "rgg":
        return inputs.rgg_laplacian(size, seed)
    return inputs.synthetic_ppt(size, seed)


def _batch(case, seed):
    """The batch's systems: each 2D or 3D with equal probability, its side
    uniform up to the case's largest. The sizes are the case's own; the seed
    gives the coefficients and right-hand sides."""
    sizes = np.random.default_rng([case["count"], case["max2d"], case["max3d"]])
    rng = np.random.default_rng(seed)
    out = []
    for k in range(case["count"]):
        two = sizes.random() < 0.5
        hi = case["max2d"] if two else case["max3d"]
        side = int(sizes.integers(min(16, hi) if two else min(8, hi), hi + 1))
        A = inputs.poisson(2 if two else 3, side, 0.5, seed * 1000 + k)
        out.append((A, rng.standard_normal(A.n)))
    return out


def _normal(seed, *shape):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    return torch.randn(*shape, dtype=torch.float64, device=DEVICE, generator=g)


def prepare(case, seed):
    if case["do"] == "batch":
        systems = _batch(case, seed)
        solver = pcg.Solver(pcg.default_config(mem_budget_mb=POOL_MB, **TYPES[case["types"]]))
        return dict(case=case, solver=solver,
                    systems=[dict(A=A, b=b, g_kind=KINDS[case["precond"]], tol=case["tol"], maxit=20000)
                             for A, b in systems])
    A = _matrix(case["system"], case["size"], seed)
    on_device = case["do"] == "construct"
    solver = pcg.Solver(pcg.default_config(g_device=int(on_device), **TYPES[case["types"]]))
    state = dict(case=case, solver=solver)
    if on_device:
        state["A"] = A
    else:
        solver.set_matrix(A)
        solver.build_precond(KINDS[case["precond"]])
    if case["do"] == "loss":
        state["w"] = _normal(seed, A.n, case["probes"])
    else:
        state["w"] = _normal(seed, A.n)
    return state


def run(state):
    case, solver = state["case"], state["solver"]
    if case["do"] == "solve":
        out = solver.solve(state["w"], tol=case["tol"], maxit=20000)
        return {"x": out.x, "iters": out.iters, "status": out.status}
    if case["do"] == "batch":
        out = solver.solve_batch(state["systems"])
        return {"x": [x for x, _ in out], "iters": np.array([r["iters"] for _, r in out], np.int64)}
    if case["do"] == "apply":
        return {"y": solver.matvec(OPS[case["op"]], state["w"])}
    if case["do"] == "loss":
        return solver.sai_loss(state["w"])
    solver.set_matrix(state["A"])
    solver.build_precond(KINDS[case["precond"]])
    return {"y": solver.matvec(pcg.OP_MINV, state["w"])}


# ------------------------------------------------------------------ the work

def _sizes(system, size):
    """(n, nonzeros of A, nonzeros of tril(A)), the graph systems' nonzeros by
    their mean."""
    if system == "poisson2d":
        n = size ** 2
        nnz = n + 4 * size * (size - 1)
    elif system == "poisson3d":
        n = size ** 3
        nnz = n + 6 * size * size * (size - 1)
    elif system == "elasticity":
        n = 3 * size ** 3
        nnz = 9 * (3 * size - 2) ** 3
    elif system == "rgg":
        n = size
        nnz = 9 * n
    else:
        n = size
        nnz = int(1.2e-3 * size * size)
    return n, nnz, (nnz + n) // 2


def _iterations(system, size, tol):
    """A nominal iteration count of FSAI-preconditioned CG, proportional to
    the digits asked for (measured: 411 on 181^2, 296 on 128^3, 98 on
    elasticity 40^3 and 1370 on P P^T of 18000 at 1e-8, 900 on a graph of
    150001 at 1e-6)."""
    base = {"poisson2d": 2.3 * size, "poisson3d": 2.34 * size, "elasticity": 2.4 * size,
            "rgg": 1200.0 * (size / 150000.0) ** 0.25, "ppt": 1370.0 * (size / 18000.0) ** 0.5}[system]
    return max(1.0, base * math.log10(1.0 / tol) / 8.0)


def work(case):
    """What one pass cannot do without. A solve or a batch: in each iteration
    the values of A and of G (G^T holds the same values) once, x, r and d read
    and written, two operations per stored entry of A, G^T and G. A product:
    the operator's values, x read, y written. The losses: A, G and the probes
    read once, three products per probe. A construction: A read, the layouts'
    values of A, G and G^T written, and the product."""
    if case["do"] == "batch":
        total = {"bytes": 0.0, "flops": 0.0}
        s2, s3 = (16 + case["max2d"]) // 2, (8 + case["max3d"]) // 2
        for system, size in (("poisson2d", s2), ("poisson3d", s3)):
            w = work(dict(case, do="solve", system=system, size=size))
            for k in total:
                total[k] += w[k] * case["count"] / 2
        return total
    ty = TYPES[case["types"]]
    sa, sg, sv = (VALUE_BYTES[ty[k]] for k in ("a_dtype", "g_dtype", "vec_dtype"))
    n, a, g = _sizes(case["system"], case["size"])
    if case["precond"] == "jacobi":
        g = n
    if case["do"] == "solve":
        it = _iterations(case["system"], case["size"], case["tol"])
        return {"bytes": it * (a * sa + g * sg + 6 * n * sv), "flops": it * (2 * a + 4 * g + 12 * n)}
    if case["do"] == "apply":
        nnz, size = {"A": (a, sa), "GT": (g, sg), "G": (g, sg), "MINV": (g, sg)}[case["op"]]
        return {"bytes": nnz * size + 16 * n, "flops": (4 if case["op"] == "MINV" else 2) * nnz}
    if case["do"] == "loss":
        k = case["probes"]
        return {"bytes": a * sa + g * sg + 8 * n * k, "flops": k * (2.0 * a + 4.0 * g + 10.0 * n)}
    return {"bytes": 12 * a + a * sa + 2 * g * sg + 16 * n, "flops": 8 * g + 4 * g}


# ------------------------------------------- the same results in plain torch

def _csr(rowptr, col, val, n):
    return torch.sparse_csr_tensor(torch.from_numpy(rowptr.astype(np.int64)), torch.from_numpy(col.astype(np.int64)),
                                   torch.from_numpy(val), size=(n, n)).to(DEVICE)


def _solution(A, b):
    """x of A x = b by Jacobi-scaled CG in FP64 to 1e-14."""
    n = A.shape[0]
    crow, col, val = A.crow_indices(), A.col_indices(), A.values()
    row = torch.repeat_interleave(torch.arange(n, device=DEVICE), crow[1:] - crow[:-1])
    dinv = torch.zeros(n, dtype=torch.float64, device=DEVICE)
    dinv[row[row == col]] = 1.0 / val[row == col]
    x = torch.zeros_like(b)
    for _ in range(2):  # the second pass starts from the true residual of the first
        r = b - A @ x
        z = dinv * r
        d = z.clone()
        rz = r @ z
        stop = 1e-14 * float(b.norm())
        for k in range(30000):
            q = A @ d
            alpha = rz / (d @ q)
            x = x + alpha * d
            r = r - alpha * q
            z = dinv * r
            new = r @ z
            if k % 50 == 49 and float(r.norm()) <= stop:
                break
            d = z + (new / rz) * d
            rz = new
    return x


def _fsai(A):
    """(G_L rows as columns, values and mask): row i of G_L solves
    A[J,J] y = e_last on J = the columns of row i up to the diagonal, scaled
    by 1 / sqrt(y_last)."""
    n = A.n
    rp = torch.from_numpy(A.rowptr.astype(np.int64)).to(DEVICE)
    col = torch.from_numpy(A.col.astype(np.int64)).to(DEVICE)
    val = torch.from_numpy(A.val).to(DEVICE)
    row = torch.repeat_interleave(torch.arange(n, device=DEVICE), rp[1:] - rp[:-1])
    key = row * n + col
    low = col <= row
    counts = torch.zeros(n, dtype=torch.int64, device=DEVICE).index_add_(0, row[low], torch.ones_like(row[low]))
    m = int(counts.max())
    J = torch.full((n, m), -1, dtype=torch.int64, device=DEVICE)
    first = torch.cumsum(counts, 0) - counts
    place = torch.arange(int(low.sum()), device=DEVICE) - first[row[low]]
    J[row[low], m - counts[row[low]] + place] = col[low]  # right-aligned: the diagonal is last
    G = torch.zeros(n, m, dtype=torch.float64, device=DEVICE)
    for i0 in range(0, n, max(1, 40_000_000 // (m * m))):
        Jc = J[i0:i0 + max(1, 40_000_000 // (m * m))]
        on = (Jc[:, :, None] >= 0) & (Jc[:, None, :] >= 0)
        want = torch.where(on, Jc[:, :, None] * n + Jc[:, None, :], torch.zeros_like(on, dtype=torch.int64))
        at = torch.searchsorted(key, want.reshape(-1)).clamp_(max=key.numel() - 1)
        S = torch.where((key[at] == want.reshape(-1)) & on.reshape(-1), val[at], torch.zeros_like(val[at])).reshape(on.shape)
        S = S + torch.diag_embed((Jc < 0).double())
        for k in range(m):  # Cholesky, column by column over all rows at once
            S[:, k, k] = torch.sqrt(S[:, k, k])
            S[:, k + 1:, k] = S[:, k + 1:, k] / S[:, k, k][:, None]
            S[:, k + 1:, k + 1:] -= S[:, k + 1:, k][:, :, None] * S[:, k + 1:, k][:, None, :]
        g = torch.zeros(S.shape[0], m, dtype=torch.float64, device=DEVICE)
        for k in range(m - 1, -1, -1):  # L^T g = e_last
            e = (S[:, k + 1:, k] * g[:, k + 1:]).sum(1)
            g[:, k] = ((1.0 if k == m - 1 else 0.0) - e) / S[:, k, k]
        G[i0:i0 + S.shape[0]] = g
    return J.clamp(min=0), torch.where(J >= 0, G, torch.zeros_like(G))


def _times_gt(F, w):
    """G^T w = G_L w, for w of shape (n,) or (n, k)."""
    J, G = F
    y = torch.zeros_like(w)
    for k in range(J.shape[1]):
        y += (G[:, k] if w.ndim == 1 else G[:, k, None]) * w[J[:, k]]
    return y


def _times_g(F, t):
    """G t = G_L^T t."""
    J, G = F
    y = torch.zeros_like(t)
    for k in range(J.shape[1]):
        y.index_add_(0, J[:, k], (G[:, k] if t.ndim == 1 else G[:, k, None]) * t)
    return y


def exact(case, seed):
    if case["do"] == "batch":  # one block-diagonal system
        systems = _batch(case, seed)
        r0 = np.cumsum([0] + [A.n for A, _ in systems])
        k0 = np.cumsum([0] + [A.nnz for A, _ in systems])
        rp = np.concatenate([[0]] + [A.rowptr[1:].astype(np.int64) + k for (A, _), k in zip(systems, k0)])
        col = np.concatenate([A.col.astype(np.int64) + r for (A, _), r in zip(systems, r0)])
        M = _csr(rp, col, np.concatenate([A.val for A, _ in systems]), int(r0[-1]))
        b = torch.from_numpy(np.concatenate([b for _, b in systems])).to(DEVICE)
        x = _solution(M, b).cpu().numpy()
        return {"x": [x[r0[k]:r0[k + 1]] for k in range(len(systems))], "iters": None}
    A = _matrix(case["system"], case["size"], seed)
    M = _csr(A.rowptr, A.col, A.val, A.n)
    if case["do"] == "solve":
        return {"x": _solution(M, _normal(seed, A.n)), "iters": None, "status": None}
    if case["do"] == "apply" and case["op"] == "A":
        return {"y": M @ _normal(seed, A.n)}
    # a plain-torch G is written for FSAI rows of grids and graphs only
    if case["precond"] != "fsai" or case["system"] == "elasticity":
        return None
    F = _fsai(A)
    if case["do"] == "loss":
        W = _normal(seed, A.n, case["probes"])
        Y = M @ _times_g(F, _times_gt(F, W))
        na = float(np.abs(A.val[A.val != 0]).mean())
        return {"sai": ((Y / na - W) ** 2).sum(0).cpu().numpy(), "l2": ((Y - W) ** 2).sum(0).cpu().numpy(),
                "cs": ((W * Y).sum(0) / (W.norm(dim=0) * Y.norm(dim=0))).cpu().numpy()}
    w = _normal(seed, A.n)
    if case["do"] == "construct" or case["op"] == "MINV":
        return {"y": _times_g(F, _times_gt(F, w))}
    return {"y": _times_gt(F, w) if case["op"] == "GT" else _times_g(F, w)}
