"""The per-tet gradient kernel against the oracle's element sums, with tet
counts below, at and past its 64 tets per workgroup and every order (row
pairs: 5, 10 and, with an odd row left over, 18)."""
import numpy as np
import pytest
import torch

import oracle
import paper_1204_2586_amd as aux
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [2, 3, 4])
@pytest.mark.parametrize("n", [1, 2, 3, 5])
def test_gradient_matches_oracle(k, n):
    xyz, tets = W.kuhn_mesh(n, 0.2 if n > 2 else 0.0, 1)
    rng = np.random.default_rng(n)
    kappa = np.exp(rng.normal(size=tets.shape[0]))
    s = aux.Solver(xyz, tets, k, kappa, device="cuda:0")
    u, lam = rng.standard_normal(s.n), rng.standard_normal(s.n)
    g = s.kappa_grad(torch.tensor(u, device="cuda:0"), torch.tensor(lam, device="cuda:0")).cpu().numpy()
    ref = oracle.Problem(xyz, tets, k, kappa).kappa_grad(u, lam)
    # sums of 35^2 terms of mixed sign, each with six rounded products
    assert np.abs(g - ref).max() <= 1e-12 * np.abs(ref).max()
