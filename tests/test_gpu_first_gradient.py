"""The first gradient of a handle that had no coefficient update uploads what it
reads and no more: the update's columns of the tet metrics come with the update."""
import numpy as np
import pytest
import torch

import oracle
import paper_1204_2586_amd as aux
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,n,nl", [(2, 6, 10), (3, 4, 20), (4, 3, 35)])
def test_first_gradient_uploads_what_it_reads(k, n, nl):
    xyz, tets = W.kuhn_mesh(n, 0.2, 1)
    rng = np.random.default_rng(k)
    nt = len(tets)
    s = aux.Solver(xyz, tets, k, device="cuda:0")
    u, lam = (torch.tensor(rng.standard_normal(s.n), device="cuda:0") for _ in range(2))
    before = int(s._info().device_bytes)
    g = s.kappa_grad(u, lam).cpu().numpy()
    # six metrics, kappa and the dofs per tet; the pair tables, twelve words for each pair of rows and column
    tables = 8 * 12 * sum(nl - 2 * m for m in range((nl + 1) // 2))
    assert int(s._info().device_bytes) - before == nt * (8 * 6 + 8 + 4 * nl) + tables
    ref = oracle.Problem(xyz, tets, k).kappa_grad(u.cpu().numpy(), lam.cpu().numpy())
    # sums of 35^2 terms of mixed sign, each with six rounded products
    assert np.abs(g - ref).max() <= 1e-12 * np.abs(ref).max()
    # the update's columns, and the gradient of the new coefficient from the same six
    kappa = np.exp(rng.normal(size=nt))
    s.set_kappa(kappa)
    fresh = aux.Solver(xyz, tets, k, kappa, device="cuda:0")
    assert torch.equal(s.kappa_grad(u, lam), fresh.kappa_grad(u, lam))
