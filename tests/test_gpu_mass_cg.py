"""The pressure mass CG on both sides of the row count where its product
stops forming the direction (32,768 rows), checked by the residual it
promises: ||r_p + M_p z_p|| <= 1e-6 ||r_p||, and the step count of a CG on
the host."""
import numpy as np
import pytest
import torch

import paper_1204_2586_amd as aux
import workloads as W

pytestmark = pytest.mark.gpu


def _steps(M, b, tol=1e-6, most=200):
    d = M.diagonal()
    r, x, k = b.copy(), np.zeros_like(b), 0
    z = r / d
    p, rz = z.copy(), r @ z
    while np.linalg.norm(r) > tol * np.linalg.norm(b) and k < most:
        q = M @ p
        a = rz / (p @ q)
        x += a * p
        r -= a * q
        z = r / d
        new = r @ z
        p = z + new / rz * p
        rz = new
        k += 1
    return k


@pytest.mark.parametrize("k,n", [(2, 1), (2, 5), (2, 31), (2, 32), (3, 15), (3, 16), (4, 3)])
def test_mass_solve(k, n):
    xyz, tets = W.kuhn_mesh(n, 0.2 if n > 2 else 0.0, 4)
    s = aux.Solver(xyz, tets, k, device="cuda:0")
    n_p = s.stokes_setup()
    M = s.export_csr("Mp")
    rng = np.random.default_rng(1)
    for scale in (1.0, 0.0, 1e-30):
        rp = scale * rng.standard_normal(n_p)
        r = torch.zeros(3 * s.n + n_p, dtype=torch.float64, device="cuda:0")
        r[3 * s.n:] = torch.tensor(rp, device="cuda:0")
        z, steps = s.stokes_qt(r)
        zp = z[3 * s.n:].cpu().numpy()
        assert np.linalg.norm(rp + M @ zp) <= 1.001e-6 * np.linalg.norm(rp)
        assert abs(steps - _steps(M, rp)) <= (1 if scale else 0)
