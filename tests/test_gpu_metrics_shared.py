"""The coefficient update and the gradient hold the tet metrics once, whichever
comes first, and agree with the oracle in both orders."""
import numpy as np
import pytest
import torch

import oracle
import paper_1204_2586_amd as aux
import workloads as W

pytestmark = pytest.mark.gpu
NLOC = {2: 10, 3: 20, 4: 35}


@pytest.mark.parametrize("k,n,operator", [(2, 8, "assembled"), (3, 5, "matfree"), (4, 4, "assembled")])
@pytest.mark.parametrize("first", ["update", "gradient"])
def test_metrics_are_held_once(k, n, operator, first):
    xyz, tets = W.kuhn_mesh(n, 0.2, 1)
    rng = np.random.default_rng(n)
    nt, nl = len(tets), NLOC[k]
    kappa = np.exp(rng.normal(size=nt))
    s = aux.Solver(xyz, tets, k, device="cuda:0", operator=operator)
    u, lam = (torch.tensor(rng.standard_normal(s.n), device="cuda:0") for _ in range(2))
    if first == "gradient":
        s.kappa_grad(u, lam)
    s.set_kappa(kappa)
    before = int(s._info().device_bytes)
    g = s.kappa_grad(u, lam).cpu().numpy()
    # the dofs by column and the pair tables (twelve words for each pair of rows and column)
    tables = 8 * 12 * sum(nl - 2 * m for m in range((nl + 1) // 2))
    assert int(s._info().device_bytes) - before == (0 if first == "gradient" else 4 * nl * nt + tables)
    p = oracle.Problem(xyz, tets, k, kappa)
    ref = p.kappa_grad(u.cpu().numpy(), lam.cpu().numpy())
    # sums of 35^2 terms of mixed sign, each with six rounded products
    assert np.abs(g - ref).max() <= 1e-12 * np.abs(ref).max()
    fresh = aux.Solver(xyz, tets, k, kappa, device="cuda:0", operator=operator)
    for what in ("A", "AH"):
        a, b = s.export_csr(what), fresh.export_csr(what)
        assert np.array_equal(a.indices, b.indices) and np.array_equal(a.data, b.data)
    if operator == "matfree":                    # its weights, too, are those of a fresh handle
        assert torch.equal(s.apply(u), fresh.apply(u))
