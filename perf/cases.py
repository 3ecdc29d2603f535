"""Workloads of the library's public entry points, for timing one build against another.

Every case is one of six kinds of call:

  matvec  y = A x with the block system of eq. 2.2 (BlockSystem.matvec)
  apply   z = M^-1 r of a preconditioner that the program keeps (BlockPreconditioner.apply)
  amg     a scalar hierarchy for a new matrix and one cycle of it (AMG, AMG.apply)
  solve   A x = b with a preconditioner that the program keeps (gmres)
  step    one step of a time or Picard loop, whose coefficients are new each time: assemble,
          build the preconditioner, solve (BlockSystem.assemble, BlockPreconditioner, gmres)
  grad    the differentiable solve and its backward pass (MGDSolve)

Inputs follow the library's synthetic workloads: diffusion coefficients that are
piecewise constant on an 8^d patch grid, 10^U(-3, 3) per patch times 10^U(-2, 2)
per group, couplings U(0.1, 10), right-hand sides U(0, 1).
"""
import torch

from paper_2002_04958_amd import api
from paper_2002_04958_amd.autograd import MGDSolve

DEV = "cuda:0"
KINDS = ("bdiag", "pctl", "schur1", "schur2", "schur2_lower")


def listed():
    return [
        # the smallest product: what a call costs besides its work
        {"name": "matvec 2D 16 G2", "call": "matvec", "dim": 2, "n": 16, "G": 2, "own": 0},
        # a program that brings its own matrices: nonsymmetric, one pattern array per block, ragged size
        {"name": "matvec 3D 41 G8 own", "call": "matvec", "dim": 3, "n": 41, "G": 8, "own": 1},
        # the product inside the largest solves
        {"name": "matvec 3D 64 G20", "call": "matvec", "dim": 3, "n": 64, "G": 20, "own": 0},
        # one application inside another program's Krylov method, default options, odd size
        {"name": "apply 2D 101 G5 schur1", "call": "apply", "dim": 2, "n": 101, "G": 5,
         "kind": "schur1", "batched": 0},
        # the same with all members batched and the launches replayed from a graph
        {"name": "apply 2D 256 G20 pctl batched", "call": "apply", "dim": 2, "n": 256, "G": 20,
         "kind": "pctl", "batched": 1},
        # the library as a scalar AMG on a large single-block matrix
        {"name": "amg 2D 1024", "call": "amg", "dim": 2, "n": 1024},
        # the smallest three-temperature solve, default options (FP64, separate launches)
        {"name": "solve 2D 64 G1 schur2", "call": "solve", "dim": 2, "n": 64, "G": 1,
         "kind": "schur2", "precision": 0, "batched": 0, "autotune": 0},
        # an ordinary twenty-group solve
        {"name": "solve 2D 256 G20 schur2 f32", "call": "solve", "dim": 2, "n": 256, "G": 20,
         "kind": "schur2", "precision": 1, "batched": 1, "autotune": 0},
        # the largest solve, as the benchmark runs it
        {"name": "solve 3D 64 G20 schur2 f32", "call": "solve", "dim": 3, "n": 64, "G": 20,
         "kind": "schur2", "precision": 1, "batched": 1, "autotune": 1},
        # a small step of a loop with new coefficients, FP64
        {"name": "step 2D 100 G4 schur2", "call": "step", "dim": 2, "n": 100, "G": 4,
         "kind": "schur2", "precision": 0, "batched": 1},
        # the largest step: setup and solve together
        {"name": "step 3D 64 G20 schur2 f32", "call": "step", "dim": 3, "n": 64, "G": 20,
         "kind": "schur2", "precision": 1, "batched": 1},
        # training through the solver: forward, adjoint and coefficient gradients
        {"name": "grad 3D 20 G3 schur2", "call": "grad", "dim": 3, "n": 20, "G": 3,
         "kind": "schur2", "precision": 0, "batched": 0},
    ]


def _log_uniform(rng, lo, hi):
    return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    call = rng.choice(("matvec", "apply", "amg", "solve", "solve", "step", "step", "grad"))
    dim = rng.choice((2, 3))
    if call == "amg":
        return {"call": call, "dim": dim,
                "n": _log_uniform(rng, 24, 1024) if dim == 2 else _log_uniform(rng, 9, 100)}
    # up to the unknowns of the largest listed cases (those of a gradient: up to a tenth)
    G = _log_uniform(rng, 1, 20)
    most = (22 * 64 ** 3 if call != "grad" else 22 * 64 ** 3 // 10) // (G + 2)
    top = min(512, int(most ** 0.5)) if dim == 2 else min(64, int(most ** (1.0 / 3.0)))
    n = _log_uniform(rng, 16, top) if dim == 2 else _log_uniform(rng, 9, top)
    case = {"call": call, "dim": dim, "n": n, "G": G}
    if call == "matvec":
        return dict(case, own=rng.choice((0, 0, 1)))
    case["kind"] = rng.choice(KINDS + ("schur2", "amg"))
    if case["kind"] == "amg" and (G + 2) * n ** dim > 1500000:
        case["kind"] = "schur2"
    case["batched"] = rng.choice((0, 1))
    if call != "apply":
        case["precision"] = rng.choice((0, 1))
    if call == "solve":
        case["autotune"] = rng.choice((0, 0, 1))
    return case


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _uniform(gen, lo, hi, *shape):
    return lo + (hi - lo) * torch.rand(*shape, dtype=torch.float64, device=DEV, generator=gen)


def _patches(dim, n):
    p = (8 * torch.arange(n, device=DEV)) // n
    idx = p
    for k in range(1, dim):
        idx = (p * 8 ** k).reshape(-1, 1) + idx.reshape(1, -1)
        idx = idx.reshape(-1)
    return idx


def _coefficients(case, seed):
    """kappa (G+2, N), c_gE, c_Eg (G, N), c_EI (N), b ((G+2) N) for one seed."""
    dim, n, G = case["dim"], case["n"], case["G"]
    N = n ** dim
    gen = torch.Generator(device=DEV).manual_seed(1000003 * (seed + 1))
    patch = _patches(dim, n)
    base = _uniform(gen, -3.0, 3.0, 8 ** dim)[patch]
    scale = _uniform(gen, -2.0, 2.0, G) if G > 1 else torch.zeros(1, dtype=torch.float64, device=DEV)
    kappa = torch.empty(G + 2, N, dtype=torch.float64, device=DEV)
    kappa[:G] = 10.0 ** (base.reshape(1, -1) + scale.reshape(-1, 1))
    kappa[G] = 10.0 ** _uniform(gen, -3.0, 3.0, 8 ** dim)[patch]
    kappa[G + 1] = 10.0 ** _uniform(gen, -3.0, 3.0, 8 ** dim)[patch]
    c_gE, c_Eg = _uniform(gen, 0.1, 10.0, G, N), _uniform(gen, 0.1, 10.0, G, N)
    c_EI = _uniform(gen, 0.1, 10.0, N)
    b = _uniform(gen, 0.0, 1.0, (G + 2) * N)
    return kappa, c_gE, c_Eg, c_EI, b, gen


def _faces(kappa, dim, n):
    """Harmonic face means, one tensor per direction: T[d][..., i] couples cell i with its
    upper neighbour in direction d (0 x, fastest)."""
    k = kappa.reshape((-1,) + (n,) * dim)
    out = []
    for d in range(dim):
        ax = dim - d  # x is the last axis
        lo, hi = k.narrow(ax, 0, n - 1), k.narrow(ax, 1, n - 1)
        out.append(2.0 * lo * hi / (lo + hi))
    return out


def _offdiag(kappa, dim, n, xi=None):
    """Off-diagonal weights (>= 0) of every row as (G+2, 2 dim, N) in the order -x +x -y +y -z +z."""
    B, N = kappa.shape[0], kappa.shape[1]
    w = torch.zeros((B, 2 * dim) + (n,) * dim, dtype=torch.float64, device=kappa.device)
    for d, T in enumerate(_faces(kappa, dim, n)):
        ax = dim - d
        w[:, 2 * d].narrow(ax, 1, n - 1).copy_(T)
        w[:, 2 * d + 1].narrow(ax, 0, n - 1).copy_(T)
    w = w.reshape(B, 2 * dim, N)
    return w if xi is None else w * (1.0 + 0.5 * xi)


def _rows(case, kappa, c_gE, c_Eg, c_EI, xi=None):
    """Off-diagonal weights and the diagonal of every block row."""
    w = _offdiag(kappa, case["dim"], case["n"], xi)
    diag = 1.0 + w.sum(1)
    G = case["G"]
    diag = torch.cat([diag[:G] + c_gE, (diag[G] + c_Eg.sum(0) + c_EI)[None],
                      (diag[G + 1] + c_EI)[None]])
    return w, diag


def _csr(w, diag, dim, n):
    """Sorted CSR arrays of one block, zero-flux neighbours left out."""
    N = n ** dim
    i = torch.arange(N, device=w.device)
    cols, vals, keep = [], [], []
    for d in reversed(range(dim)):  # -z -y -x, the diagonal, +x +y +z: ascending columns
        cols.append(i - n ** d)
        vals.append(-w[2 * d])
        keep.append((i // n ** d) % n > 0)
    cols.append(i)
    vals.append(diag)
    keep.append(torch.ones_like(i, dtype=torch.bool))
    for d in range(dim):
        cols.append(i + n ** d)
        vals.append(-w[2 * d + 1])
        keep.append((i // n ** d) % n < n - 1)
    cols, vals, keep = (torch.stack(t, 1) for t in (cols, vals, keep))
    rp = torch.zeros(N + 1, dtype=torch.int32, device=w.device)
    rp[1:] = keep.sum(1).cumsum(0)
    return rp, cols[keep].to(torch.int32), vals[keep].contiguous()


def _system(ctx, case, seed):
    kappa, c_gE, c_Eg, c_EI, b, gen = _coefficients(case, seed)
    dim, n, G = case["dim"], case["n"], case["G"]
    N = n ** dim
    if case.get("own"):
        xi = _uniform(gen, 0.0, 1.0, G + 2, 2 * dim, N)
        w, diag = _rows(case, kappa, c_gE, c_Eg, c_EI, xi)
        blocks = [_csr(w[a], diag[a], dim, n) for a in range(G + 2)]
        return api.BlockSystem.from_tensors(ctx, G, N, blocks, -c_gE, -c_Eg, -c_EI, -c_EI), b
    co = api.Coeffs(dim, n, G, kappa.reshape(-1), c_gE.reshape(-1), c_Eg.reshape(-1), c_EI)
    return api.BlockSystem.assemble(ctx, co), b


def _options(case):
    out = {"batched": case["batched"], "use_graph": case["batched"]}
    if case.get("precision"):
        out["amg_precision"] = 1
    if case.get("autotune"):
        out["amg_autotune"] = 1
    return out


def prepare(case, seed):
    call = case["call"]
    if call == "amg":
        gen = torch.Generator(device=DEV).manual_seed(1000003 * (seed + 1))
        dim, n = case["dim"], case["n"]
        kappa = 10.0 ** _uniform(gen, -3.0, 3.0, 1, 8 ** dim)[:, _patches(dim, n)]
        w = _offdiag(kappa, dim, n)
        rp, ci, v = _csr(w[0], 1.0 + w[0].sum(0), dim, n)
        r = _uniform(gen, 0.0, 1.0, n ** dim)
        return {"call": call, "ctx": api.Context(0), "rp": rp, "ci": ci, "v": v, "r": r}
    if call == "grad":
        kappa, c_gE, c_Eg, c_EI, b, gen = _coefficients(case, seed)
        leaves = [t.requires_grad_(True) for t in (kappa, c_gE, c_Eg, c_EI, b)]
        gx = _uniform(gen, 0.0, 1.0, b.numel())
        return {"call": call, "leaves": leaves, "gx": gx, "case": case, "options": _options(case)}
    ctx = api.Context(0)
    if call == "step":
        kappa, c_gE, c_Eg, c_EI, b, _ = _coefficients(case, seed)
        return {"call": call, "ctx": ctx, "case": case, "b": b, "options": _options(case),
                "kappa": kappa.reshape(-1), "c_gE": c_gE.reshape(-1), "c_Eg": c_Eg.reshape(-1),
                "c_EI": c_EI}
    system, b = _system(ctx, case, seed)
    state = {"call": call, "ctx": ctx, "system": system, "b": b}
    if call == "matvec":
        state["y"] = torch.empty_like(b)
    else:
        state["M"] = api.BlockPreconditioner(ctx, system, case["kind"], **_options(case))
        if call == "apply":
            state["z"] = torch.empty_like(b)
    return state


def run(s):
    call = s["call"]
    if call == "matvec":
        return s["system"].matvec(s["b"], s["y"])
    if call == "apply":
        return s["M"].apply(s["b"], s["z"])
    if call == "solve":
        return api.gmres(s["ctx"], s["system"], s["M"], s["b"], rtol=1e-8)[0]
    if call == "amg":
        h = api.AMG(s["ctx"], s["rp"], s["ci"], s["v"])
        z = h.apply(s["r"])
        h.close()
        return z
    c = s["case"]
    if call == "step":
        co = api.Coeffs(c["dim"], c["n"], c["G"], s["kappa"], s["c_gE"], s["c_Eg"], s["c_EI"])
        system = api.BlockSystem.assemble(s["ctx"], co)
        M = api.BlockPreconditioner(s["ctx"], system, c["kind"], **s["options"])
        x = api.gmres(s["ctx"], system, M, s["b"], rtol=1e-8)[0]
        M.close()
        system.close()
        return x
    x = MGDSolve.apply(*s["leaves"], c["dim"], c["n"], c["kind"], 1e-8, s["options"])
    grads = torch.autograd.grad(x, s["leaves"], s["gx"])
    return [x.detach()] + list(grads)


def work(case):
    """Inputs read once, outputs written once; two operations per matrix entry and coupling."""
    dim, N = case["dim"], case["n"] ** case["dim"]
    nnz = N * (2 * dim + 1)
    if case["call"] == "amg":
        return {"bytes": 12.0 * nnz + 4.0 * N + 16.0 * N, "flops": 2.0 * nnz}
    G = case["G"]
    B, couplings = G + 2, 2 * G + 2
    flops = 2.0 * N * (B * (2 * dim + 1) + couplings)
    coeffs = 8.0 * N * (B + 2 * G + 1)
    if case["call"] == "step":
        return {"bytes": coeffs + 16.0 * B * N, "flops": flops}
    if case["call"] == "grad":
        return {"bytes": 2.0 * coeffs + 32.0 * B * N, "flops": 2.0 * flops}
    # one pattern, one value per entry of every block, the couplings, x and y
    pattern = (4.0 * nnz + 4.0 * N) * (B if case.get("own") else 1)
    return {"bytes": pattern + 8.0 * B * nnz + 8.0 * couplings * N + 16.0 * B * N, "flops": flops}


# ---------------------------------------------------------------------------
# the same values in plain torch, 64 bits
# ---------------------------------------------------------------------------
DENSE_MOST = 13000  # unknowns of a system that a dense factorisation solves in seconds


def _product(case, w, diag, c_gE, c_Eg, c_EI, x):
    dim, n, G = case["dim"], case["n"], case["G"]
    X = x.reshape((G + 2,) + (n,) * dim)
    W = w.reshape((G + 2, 2 * dim) + (n,) * dim)
    y = diag.reshape(X.shape) * X
    for d in range(dim):
        ax = dim - d
        lo, hi = X.narrow(ax, 0, n - 1), X.narrow(ax, 1, n - 1)
        y.narrow(ax, 1, n - 1).sub_(W[:, 2 * d].narrow(ax, 1, n - 1) * lo)
        y.narrow(ax, 0, n - 1).sub_(W[:, 2 * d + 1].narrow(ax, 0, n - 1) * hi)
    x, y = x.reshape(G + 2, -1), y.reshape(G + 2, -1)
    y[:G] -= c_gE * x[G]
    y[G] -= (c_Eg * x[:G]).sum(0) + c_EI * x[G + 1]
    y[G + 1] -= c_EI * x[G]
    return y.reshape(-1)


def _dense(case, w, diag, c_gE, c_Eg, c_EI):
    dim, n, G = case["dim"], case["n"], case["G"]
    N = n ** dim
    A = torch.zeros((G + 2) * N, (G + 2) * N, dtype=torch.float64, device=w.device)
    i = torch.arange(N, device=w.device)
    for a in range(G + 2):
        r = a * N + i
        A[r, r] = diag[a]
        for d in range(dim):
            at = (i // n ** d) % n
            lo, hi = i[at > 0], i[at < n - 1]
            A[a * N + lo, a * N + lo - n ** d] = -w[a, 2 * d][lo]
            A[a * N + hi, a * N + hi + n ** d] = -w[a, 2 * d + 1][hi]
    for g in range(G):
        A[g * N + i, G * N + i] = -c_gE[g]
        A[G * N + i, g * N + i] = -c_Eg[g]
    A[G * N + i, (G + 1) * N + i] = -c_EI
    A[(G + 1) * N + i, G * N + i] = -c_EI
    return A


def _refined(solve, A, b):
    """A solution of A x = b with two steps of refinement."""
    x = solve(b)
    for _ in range(2):
        x = x + solve(b - A @ x)
    return x


def exact(case, seed):
    call = case["call"]
    if call in ("apply", "amg"):
        return None  # a V-cycle has no value apart from the method itself
    kappa, c_gE, c_Eg, c_EI, b, gen = _coefficients(case, seed)
    xi = None
    if case.get("own"):
        xi = _uniform(gen, 0.0, 1.0, case["G"] + 2, 2 * case["dim"], case["n"] ** case["dim"])
    if call == "matvec":
        w, diag = _rows(case, kappa, c_gE, c_Eg, c_EI, xi)
        return _product(case, w, diag, c_gE, c_Eg, c_EI, b)
    if b.numel() > DENSE_MOST:
        return None
    w, diag = _rows(case, kappa, c_gE, c_Eg, c_EI)
    A = _dense(case, w, diag, c_gE, c_Eg, c_EI)
    lu = torch.linalg.lu_factor(A)
    x = _refined(lambda r: torch.linalg.lu_solve(*lu, r.reshape(-1, 1)).reshape(-1), A, b)
    if call != "grad":
        return x
    gx = _uniform(gen, 0.0, 1.0, b.numel())
    At = A.t().contiguous()
    lut = torch.linalg.lu_factor(At)
    lam = _refined(lambda r: torch.linalg.lu_solve(*lut, r.reshape(-1, 1)).reshape(-1), At, gx)
    # the gradient of -lam . (A(kappa, c) x) with lam and x held
    leaves = [t.detach().clone().requires_grad_(True) for t in (kappa, c_gE, c_Eg, c_EI)]
    k, gE, Eg, EI = leaves
    G, X, Lm = case["G"], x.reshape(case["G"] + 2, -1), lam.reshape(case["G"] + 2, -1)
    total = (Lm[:G] * gE * (X[:G] - X[G])).sum() + (Lm[G] * Eg * (X[G] - X[:G])).sum()
    total = total + ((Lm[G] - Lm[G + 1]) * EI * (X[G] - X[G + 1])).sum()
    dim, n = case["dim"], case["n"]
    Xn, Ln = (t.reshape((-1,) + (n,) * dim) for t in (X, Lm))
    for d, T in enumerate(_faces(k, dim, n)):
        ax = dim - d
        dx = Xn.narrow(ax, 0, n - 1) - Xn.narrow(ax, 1, n - 1)
        dl = Ln.narrow(ax, 0, n - 1) - Ln.narrow(ax, 1, n - 1)
        total = total + (T * dx * dl).sum()
    return [x] + [-g for g in torch.autograd.grad(total, leaves)] + [lam]
