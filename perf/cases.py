"""Timed cases of the solver: the calls that programs make, over the sizes they make them at.

Every problem is -div(kappa grad u) = f on the unit cube (n^3 cubes of six
tetrahedra, the interior vertices moved by up to ``jitter`` mesh widths), in
P^k elements, through the public entry points of ``paper_1204_2586_amd``.
``prepare`` sets up the handle that such a program keeps and its vectors on
the GPU, all from the seed: another seed is another mesh jitter, another
coefficient field and other vectors.  ``exact`` solves the same problem by
itself: element matrices from exact monomial integrals, one sparse matrix,
conjugate gradients with a diagonal preconditioner to rounding.

Kinds of calls:

* ``solve``      one CG solve, the main use;
* ``apply``      one application of the preconditioner, as a program with a Krylov method of its own calls it;
* ``fgmres``     one FGMRES(30) solve, the Krylov method of the paper's experiments;
* ``batched``    nrhs sources solved in lock-step;
* ``block``      the same sources by block CG;
* ``stokes``     one FGMRES solve of the Hood-Taylor Stokes system with the block triangular preconditioner;
* ``adjoint``    two steps of a coefficient identification: for each of two trial fields log kappa a coefficient
                 update, the forward solve, the adjoint solve and the gradient, through the autograd function;
* ``matvec``     one product with A_h;
* ``kappa_grad`` the per-tet gradient alone.
"""
import math

import numpy as np
import torch

import paper_1204_2586_amd as aux


def _case(name, kind, order, n, jitter=0.2, grf=False, precision="fp64", operator="assembled", aux_space=1, nrhs=1,
          tol=1e-8):
    c = dict(kind=kind, order=order, n=n, jitter=jitter, grf=grf, precision=precision, operator=operator,
             aux_space=aux_space, nrhs=nrhs, tol=tol)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: one application inside somebody else's Krylov loop, 3,375 unknowns; launches count
        _case("apply_p2_n8", "apply", 2, 8),
        # a small whole solve in the default precision, odd size, rough coefficient: one of many in a parameter study
        _case("solve_p2_n13_grf", "solve", 2, 13, jitter=0.0, grf=True),
        # the benchmark's headline: 857,375 unknowns, FP32 preconditioner inside FP64 CG
        _case("solve_p2_n48_jitter", "solve", 2, 48, precision="mixed"),
        # the benchmark's high-order matrix-free solve with a rough coefficient, at the same number of unknowns
        _case("solve_p3_n32_grf_matfree", "solve", 3, 32, jitter=0.0, grf=True, precision="mixed", operator="matfree"),
        # order 4 with the intermediate P2 space, everything in FP64; the P4 operator assembled
        _case("solve_p4_n14_grf_nested", "solve", 4, 14, jitter=0.0, grf=True, aux_space=2),
        # many sources on one mesh: 32 columns, the largest amount of work here
        _case("batched_p2_n40_rhs32", "batched", 2, 40, jitter=0.0, precision="mixed", nrhs=32),
        # a few sources at an odd width (padded inside) and order 3, in FP64
        _case("batched_p3_n15_rhs5", "batched", 3, 15, nrhs=5),
        # the paper's Krylov method on a mesh of odd size
        _case("fgmres_p2_n33_jitter", "fgmres", 2, 33),
        # the paper's second test problem, P2-P1
        _case("stokes_p2p1_n20_jitter", "stokes", 2, 20),
        # coefficient identification: updates, forward and adjoint solves, gradients
        _case("adjoint_p2_n32_grf", "adjoint", 2, 32, jitter=0.0, grf=True, precision="mixed", tol=1e-10),
        # the operator alone, order 3, odd size
        _case("matvec_p3_n25_jitter", "matvec", 3, 25),
        # the gradient alone, order 3
        _case("kappa_grad_p3_n24_grf", "kappa_grad", 3, 24, jitter=0.0, grf=True),
    ]


# the largest n that a drawn case of a kind has, by order: no more work than the listed cases have
_MOST = {
    "apply": {2: 40, 3: 27, 4: 20}, "solve": {2: 40, 3: 26, 4: 18}, "fgmres": {2: 33, 3: 20, 4: 14},
    "batched": {2: 32, 3: 20, 4: 12}, "block": {2: 28, 3: 16, 4: 10}, "stokes": {2: 20, 3: 10},
    "adjoint": {2: 28, 3: 16, 4: 10}, "matvec": {2: 40, 3: 26, 4: 18}, "kappa_grad": {2: 40, 3: 26, 4: 18},
}


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "apply", "fgmres", "batched", "block", "stokes", "adjoint", "matvec",
                       "kappa_grad"])
    order = rng.choice(sorted(_MOST[kind]))
    n = _log_uniform(rng, 6 if order == 2 else 4, _MOST[kind][order])
    grf = rng.random() < 0.5
    jitter = 0.0 if grf else rng.choice([0.0, round(rng.uniform(0.05, 0.2), 3)])
    # one application in FP32 is left out: nothing corrects its rounding
    precision = "fp64" if kind in ("apply", "fgmres", "stokes") else rng.choice(["fp64", "mixed"])
    operator = "assembled" if kind in ("batched", "block", "stokes") else rng.choice(["assembled", "matfree"])
    aux_space = rng.choice([1, 2]) if kind in ("solve", "apply") and order > 2 else 1
    nrhs = 1
    if kind in ("batched", "block"):
        most = min(64 if kind == "batched" else 8, 15_000_000 // (order * n - 1) ** 3)
        nrhs = _log_uniform(rng, 2, max(2, most))
        grf = False
    tol = 1e-10 if kind == "adjoint" else 1e-8
    return _case(None, kind, order, n, jitter, grf, precision, operator, aux_space, nrhs, tol)


# ---------------------------------------------------------------- inputs

_AXES = [(0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0)]


def _mesh(n, jitter, seed):
    """Vertices [nv, 3] and tets [6 n^3, 4] of the unit cube, as numpy arrays."""
    m = n + 1
    g = np.indices((m, m, m)).reshape(3, -1).T
    xyz = g / n
    inside = np.all((g > 0) & (g < n), axis=1)
    if jitter:
        move = np.random.default_rng(seed).uniform(-jitter / n, jitter / n, size=(int(inside.sum()), 3))
        xyz[inside] += move
    cube = np.indices((n, n, n)).reshape(3, -1).T
    tets = np.empty((n ** 3, 6, 4), dtype=np.int32)
    for s, axes in enumerate(_AXES):
        p = cube.copy()
        for v in range(4):
            if v:
                p[:, axes[v - 1]] += 1
            tets[:, s, v] = (p[:, 0] * m + p[:, 1]) * m + p[:, 2]
    return xyz, tets.reshape(-1, 4)


def _log_kappa(xyz, tets, seed, sigma=2.3, ell=0.1, features=512):
    """A smooth Gaussian random field at the tets' centroids (device tensor)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    kw = dict(generator=g, device="cuda", dtype=torch.float64)
    w = torch.randn(3, features, **kw) / ell
    b = torch.rand(features, **kw) * (2 * math.pi)
    x = torch.tensor(xyz, device="cuda")
    c = x[torch.tensor(tets, device="cuda").long()].mean(1)
    return sigma * math.sqrt(2.0 / features) * torch.cat([torch.cos(p @ w + b).sum(1) for p in c.split(1 << 17)])


def _nodes(order):
    """Barycentric multi-indices of a tet's P^k nodes."""
    r = range(order + 1)
    return [(a, b, c, order - a - b - c) for a in r for b in r for c in r if a + b + c <= order]


def _space(xyz, tets, order):
    """The P^k space without its boundary nodes, numbered by the sorted vertex
    ids of each node: (dof of each tet's nodes [nt, nloc], -1 on the boundary,
    and the positions [n_h, 3]), on the device."""
    t = torch.tensor(tets, device="cuda").long()
    nv = xyz.shape[0]
    keys = []
    for alpha in _nodes(order):
        ids = torch.stack([t[:, v] for v in range(4) for _ in range(alpha[v])], 1).sort(1).values
        k = torch.zeros_like(ids[:, 0])
        for j in range(order):
            k = k * nv + ids[:, j]
        keys.append(k)
    uniq, inv = torch.unique(torch.stack(keys, 1), return_inverse=True)
    x = torch.tensor(xyz, device="cuda")
    low = torch.ones(uniq.shape[0], 3, dtype=torch.bool, device="cuda")
    high, pos, k = low.clone(), torch.zeros(uniq.shape[0], 3, dtype=torch.float64, device="cuda"), uniq
    for _ in range(order):
        v = x[k % nv]
        low &= v == 0.0
        high &= v == 1.0
        pos += v / order
        k = k // nv
    inside = ~(low | high).any(1)
    number = torch.where(inside, inside.long().cumsum(0) - 1, -1)
    return number[inv], pos[inside]


def _source(pos, h, seed, columns, modes=16, kmax=4):
    """Values of random smooth sources at the nodes, times the cell volume: [n_h, columns]."""
    rng = np.random.default_rng(1000 + seed)
    amp = torch.tensor(rng.normal(size=(kmax ** 3, columns)) * (rng.random((kmax ** 3, columns)) < modes / kmax ** 3)
                       + 0.1, device="cuda")
    k = torch.arange(1, kmax + 1, device="cuda", dtype=torch.float64)
    s = [torch.sin(math.pi * pos[:, a:a + 1] * k) for a in range(3)]
    wave = (s[0][:, :, None, None] * s[1][:, None, :, None] * s[2][:, None, None, :]).reshape(pos.shape[0], -1)
    return (wave @ amp) * h ** 3


def _problem(case, seed):
    xyz, tets = _mesh(case["n"], case["jitter"], seed)
    lk = _log_kappa(xyz, tets, seed) if case["grf"] or case["kind"] == "adjoint" else None
    dofs, pos = _space(xyz, tets, case["order"])
    return xyz, tets, lk, dofs, pos


def _vectors(case, seed, pos, n_tets):
    """The call's vectors on the device."""
    n, kind = pos.shape[0], case["kind"]
    g = torch.Generator(device="cuda").manual_seed(seed + 77)
    noise = lambda: torch.randn(n, generator=g, device="cuda", dtype=torch.float64)  # noqa: E731
    if kind in ("apply", "matvec"):
        return dict(x=noise())
    if kind == "kappa_grad":
        s = _source(pos, 1.0, seed, 2)
        return dict(u=s[:, 0] + 0.01 * noise(), lam=s[:, 1] + 0.01 * noise())
    if kind == "stokes":
        return dict(f=_source(pos, 1.0 / case["n"], seed, 3))
    b = _source(pos, 1.0 / case["n"], seed, case["nrhs"])
    if kind == "adjoint":
        return dict(f=b[:, 0].contiguous(), want=1e-2 * _source(pos, 1.0, seed + 5, 1)[:, 0])
    return dict(f=b.contiguous() if kind in ("batched", "block") else b[:, 0].contiguous())


def prepare(case, seed):
    xyz, tets, lk, dofs, pos = _problem(case, seed)
    state = _vectors(case, seed, pos, tets.shape[0])
    state.update(kind=case["kind"], tol=case["tol"])
    opts = dict(precision=case["precision"], operator=case["operator"], aux_space=case["aux_space"], device="cuda:0")
    if case["kind"] == "adjoint":
        # the field of the last accepted step, then two trial fields near it
        step = _log_kappa(xyz, tets, seed + 1)
        state["problem"] = aux.KappaSolve(xyz, tets, case["order"], tol=case["tol"], **opts)
        state["trials"] = [(lk + 0.1 * step).contiguous(), (lk - 0.1 * step).contiguous()]
        state["problem"].solver_for(torch.exp(lk).cpu().numpy())
        return state
    s = aux.Solver(xyz, tets, case["order"], None if lk is None else torch.exp(lk).cpu().numpy(), **opts)
    state["solver"] = s
    if case["kind"] == "stokes":
        n_p = s.stokes_setup()
        f = state.pop("f")
        state["f"] = torch.cat([f.T.reshape(-1), torch.zeros(n_p, dtype=torch.float64, device="cuda")])
    return state


def run(state):
    kind = state["kind"]
    if kind == "adjoint":
        out = []
        for trial in state["trials"]:
            f = state["f"].detach().requires_grad_()
            lk = trial.detach().requires_grad_()
            u = aux.AuxSolveFn.apply(f, lk, state["problem"])
            (0.5 * (u - state["want"]).square().sum()).backward()
            out.append((u.detach(), f.grad, lk.grad))
        return out
    s, tol = state["solver"], state["tol"]
    if kind == "apply":
        return s.apply(state["x"])
    if kind == "matvec":
        return s.matvec(state["x"])
    if kind == "kappa_grad":
        return s.kappa_grad(state["u"], state["lam"])
    if kind == "fgmres":
        return s.fgmres(state["f"], tol=tol)[0]
    if kind == "stokes":
        return s.stokes_fgmres(state["f"], tol=tol)[0]
    if kind == "batched":
        return s.solve_batched(state["f"], tol=tol)[0]
    if kind == "block":
        return s.solve_block(state["f"], tol=tol)[0]
    return s.solve(state["f"], tol=tol)[0]


# ---------------------------------------------------------------- needed work

_ROW = {2: 28, 3: 45, 4: 70}          # entries of A_h per row
_STEPS = {2: 24, 3: 30, 4: 40}        # CG steps with the P^1 space


def work(case):
    """Bytes and operations of one pass: per step the FP64 product, the four
    P^k products of the two-sweep smoother and the vectors once, the matrix
    values at their width with no index, every column sharing them."""
    k, n, kind, m = case["order"], case["n"], case["kind"], case["nrhs"]
    rows, tets = (k * n - 1) ** 3, 6 * n ** 3
    nnz, nloc = rows * _ROW[k], math.comb(k + 3, 3)
    s = 4 if case["precision"] == "mixed" else 8
    if case["operator"] == "matfree":
        # node numbers, six weights and the coefficient's share per tet; element products
        product = lambda w: (tets * (4 * nloc + 6 * w), tets * (6 * nloc * nloc + 2 * nloc * nloc))  # noqa: E731
    else:
        product = lambda w: (nnz * w, 2 * nnz)  # noqa: E731
    if kind == "matvec":
        return dict(bytes=nnz * 8 + 16 * rows, flops=2 * nnz)
    if kind == "kappa_grad":
        return dict(bytes=tets * (4 * nloc + 7 * 8 + 8) + 16 * rows, flops=tets * (12 * nloc * nloc))
    b, f = product(s)
    apply = (4 * b + m * 16 * rows, 4 * f * m)
    if kind == "apply":
        return dict(bytes=apply[0], flops=apply[1])
    b, f = product(8)
    step = (apply[0] + b + m * 40 * rows, apply[1] + f * m)
    steps = _STEPS[k]
    if kind == "stokes":
        # three velocity components a step, their products and the divergence block
        return dict(bytes=50 * (3 * step[0] + 8 * nnz), flops=50 * (3 * step[1] + 2 * nnz))
    if kind == "adjoint":
        # per trial field two solves, the operator's values written once and the gradient
        return dict(bytes=2 * (2 * steps * step[0] + 16 * nnz + tets * 8), flops=2 * 2 * steps * step[1])
    if case["aux_space"] == 2:
        steps = 0.7 * steps
    return dict(bytes=steps * step[0], flops=steps * step[1])


# ---------------------------------------------------------------- exact values

def _reference(order):
    """R[i, j, a, b] = integral over the reference tet of d_i phi_a d_j phi_b."""
    nodes = np.array(_nodes(order), dtype=np.float64)[:, 1:] / order
    powers = [(i, j, l) for i in range(order + 1) for j in range(order + 1 - i) for l in range(order + 1 - i - j)]
    coef = np.linalg.inv(np.stack([np.prod(nodes ** np.array(p), axis=1) for p in powers], 1))     # [monomial, node]
    fact = math.factorial
    R = np.zeros((3, 3, len(powers), len(powers)))
    for a, p in enumerate(powers):
        for b, q in enumerate(powers):
            for i in range(3):
                for j in range(3):
                    if p[i] and q[j]:
                        e = [p[v] + q[v] - (v == i) - (v == j) for v in range(3)]
                        R[i, j, a, b] = p[i] * q[j] * math.prod(map(fact, e)) / fact(sum(e) + 3)
    return np.einsum("ijpq,pa,qb->ijab", R, coef, coef)


def _element_matrices(xyz, tets, order, kappa):
    """[nt, nloc, nloc] element stiffness matrices on the device."""
    x = torch.tensor(xyz, device="cuda")[torch.tensor(tets, device="cuda").long()]
    # reference coordinate i belongs to vertex 1 + i
    J = torch.stack([x[:, v] - x[:, 0] for v in (1, 2, 3)], 2)
    e = [J[:, :, v] for v in range(3)]
    det = (e[0] * torch.linalg.cross(e[1], e[2])).sum(1)
    inv = torch.stack([torch.linalg.cross(e[1], e[2]), torch.linalg.cross(e[2], e[0]),
                       torch.linalg.cross(e[0], e[1])], 1) / det[:, None, None]
    G = (inv[:, :, None, :] * inv[:, None, :, :]).sum(3) * det.abs()[:, None, None]
    if kappa is not None:
        G = G * kappa[:, None, None]
    R = torch.tensor(_reference(order), device="cuda")
    nloc = R.shape[2]
    return (G.reshape(-1, 9) @ R.reshape(9, -1)).reshape(-1, nloc, nloc)


def _assemble(K, dofs, n):
    nloc = dofs.shape[1]
    row = dofs[:, :, None].expand(-1, -1, nloc).reshape(-1)
    col = dofs[:, None, :].expand(-1, nloc, -1).reshape(-1)
    keep = (row >= 0) & (col >= 0)
    A = torch.sparse_coo_tensor(torch.stack([row[keep], col[keep]]), K.reshape(-1)[keep], (n, n)).coalesce()
    return A.to_sparse_csr(), torch.zeros(n, dtype=torch.float64, device="cuda").index_add_(
        0, dofs[dofs >= 0], K.diagonal(dim1=1, dim2=2)[dofs >= 0])


def _cg(A, diag, B, rtol=1e-14, most=6000):
    """A^{-1} B for a block of columns, each by its own CG with the diagonal preconditioner, then one correction
    with the residual of the result."""
    X = torch.zeros_like(B)
    for _ in range(2):
        R = B - A @ X
        D, Z = torch.zeros_like(X), R / diag[:, None]
        P, rz = Z.clone(), (R * Z).sum(0)
        stop = (rz * rtol ** 2).clamp_min(1e-300)
        for k in range(most):
            Q = A @ P
            alpha = rz / (P * Q).sum(0).clamp_min(1e-300)
            D += alpha * P
            R -= alpha * Q
            Z = R / diag[:, None]
            new = (R * Z).sum(0)
            P = Z + (new / rz.clamp_min(1e-300)) * P
            rz = new
            if k % 25 == 24 and bool((rz <= stop).all()):
                break
        X += D
        rtol = 1e-6
    return X


def exact(case, seed):
    kind = case["kind"]
    if kind in ("apply", "stokes"):
        # the preconditioner has no value apart from the hierarchy that the library builds; the saddle-point
        # system takes too long without a preconditioner
        return None
    xyz, tets, lk, dofs, pos = _problem(case, seed)
    v = _vectors(case, seed, pos, tets.shape[0])
    n = pos.shape[0]
    if kind == "adjoint":
        step, out = _log_kappa(xyz, tets, seed + 1), []
        for trial in (lk + 0.1 * step, lk - 0.1 * step):
            K = _element_matrices(xyz, tets, case["order"], torch.exp(trial))
            A, diag = _assemble(K, dofs, n)
            u = _cg(A, diag, v["f"][:, None])[:, 0]
            lam = _cg(A, diag, (u - v["want"])[:, None])[:, 0]
            out.append((u, lam, _gradient(K, dofs, u, lam)))
        return out
    K = _element_matrices(xyz, tets, case["order"], None if lk is None else torch.exp(lk))
    if kind == "kappa_grad":
        return _gradient(K, dofs, v["u"], v["lam"])
    A, diag = _assemble(K, dofs, n)
    if kind == "matvec":
        return (A @ v["x"][:, None])[:, 0]
    f = v["f"] if v["f"].dim() == 2 else v["f"][:, None]
    x = _cg(A, diag, f)
    return x if v["f"].dim() == 2 else x[:, 0]


def _gradient(K, dofs, u, lam):
    at = dofs.clamp_min(0)
    ue, le = (torch.where(dofs >= 0, w[at], 0.0) for w in (u, lam))
    return -(le[:, :, None] * K * ue[:, None, :]).sum((1, 2))
