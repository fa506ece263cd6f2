"""Meshes whose vertices and tets are numbered without regard to their places:
slices of A_h with 32-bit columns by need beside 16-bit ones, tiles and patches
whose dofs are far apart in memory, compared with the host's matrix, with each
other and (small) with the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_1204_2586_amd as aux
import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _mesh(n, share, seed):
    """A cube mesh with `share` of its vertex ids exchanged among themselves and the tets in any order."""
    xyz, tets = W.kuhn_mesh(n, 0.2, seed)
    rng = np.random.default_rng(seed)
    some = np.flatnonzero(rng.random(len(xyz)) < share)
    to = np.arange(len(xyz))
    to[some] = rng.permutation(some)
    out = np.empty_like(xyz)
    out[to] = xyz
    return out, np.ascontiguousarray(to[tets][rng.permutation(len(tets))].astype(np.int32))


def _rel(a, b):
    return float((a - b).norm() / b.norm())


@pytest.mark.parametrize("k,n,share", [(2, 24, 0.05), (2, 24, 1.0), (3, 18, 1.0), (4, 6, 1.0)])
def test_renumbered_mesh(k, n, share):
    """The FP64 product within the bound of sums of at most 400 terms, operator
    forms and block layouts as in their tests on cube numbering (1e-12 and 2e-6
    for one application, 1e-10 and 1e-5 after three steps)."""
    xyz, tets = _mesh(n, share, 3)
    s = aux.Solver(xyz, tets, k, device=DEV, sell_window=4096)
    per_entry = s.info.sell_index_bytes / s.info.stored_A
    print(f"[renumbered k={k} n={n} share={share}] column bytes per entry {per_entry:.3f}", flush=True)
    if n >= 18:
        assert 2.125 < per_entry < 4.0                    # both forms
    rng = np.random.default_rng(1)
    x = torch.tensor(rng.standard_normal(s.n), device=DEV)
    ref = torch.tensor(s.export_csr("A") @ x.cpu().numpy(), device=DEV)
    assert _rel(s.matvec(x), ref) <= 400 * 2.0 ** -53
    for prec, tol in (("fp64", 1e-12), ("mixed", 2e-6)):
        s.set_precision(prec)
        z = s.apply(x)
        s.set_operator("matfree")
        assert _rel(s.apply(x), z) <= tol, prec
        s.set_operator("assembled")
    nrhs = 16
    F = torch.tensor(rng.standard_normal((s.n, nrhs)), device=DEV)
    a, b = (aux.Solver(xyz, tets, k, device=DEV, batch_tiles=t) for t in (2, 0))
    for prec, tol in (("fp64", 1e-10), ("mixed", 1e-5)):
        out = []
        for h in (a, b):
            h.set_precision(prec)
            out.append(h.solve_batched(F, tol=0.0, maxit=3, check=False)[0])
        assert min(a.info.batch_tile_rows) > 0
        assert _rel(out[0], out[1]) <= tol, prec


@pytest.mark.parametrize("k,n", [(2, 6), (3, 5), (4, 3)])
def test_renumbered_mesh_matches_oracle(k, n):
    """One application and the CG iterates, both operators, as on cube numbering."""
    xyz, tets = _mesh(n, 1.0, 2)
    s = aux.Solver(xyz, tets, k, device=DEV)
    o = oracle.Problem(xyz, tets, k).setup_amg()
    r, b = W.random_vector(s.n, 4), o.load(W.manufactured_f)
    want, x = o.apply(r), o.pcg(b, tol=0.0, maxit=5)[0]
    for op in ("assembled", "matfree"):
        s.set_operator(op)
        z = s.apply(torch.tensor(r, device=DEV)).cpu().numpy()
        assert np.linalg.norm(z - want) <= 1e-12 * np.linalg.norm(want), op
        u = s.solve(torch.tensor(b, device=DEV), tol=0.0, maxit=5, check=False)[0].cpu().numpy()
        assert np.linalg.norm(u - x) <= 1e-10 * np.linalg.norm(x), op
