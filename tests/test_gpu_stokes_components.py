"""The velocity block of the Stokes operator and of Q_t, three components at
once or one by one (by the handle's options): with a zero pressure part each
component is what the scalar product or preconditioner gives."""
import numpy as np
import pytest
import torch

import paper_1204_2586_amd as aux
import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-13), ("mixed", 1e-6)])
@pytest.mark.parametrize("k,n,opts", [
    (2, 1, {}), (2, 2, {}), (2, 9, {}), (2, 9, dict(operator="matfree")), (2, 9, dict(fuse_cycle=False)),
    (2, 9, dict(cycle_lanes=4)), (2, 9, dict(cycle_lanes=-8, dense_cycle_rows=0, nu=1)), (2, 21, {}),
    (3, 7, dict(aux_space=2)), (3, 7, dict(nu=3, sell_index16=False)), (4, 5, {})])
def test_components_equal_scalar_calls(k, n, opts, precision, tol):
    xyz, tets = W.kuhn_mesh(n, 0.2 if n > 2 else 0.0, 1)
    s = aux.Solver(xyz, tets, k, device=DEV, precision=precision, sell_window=1 << 30, **opts)
    n_p = s.stokes_setup()
    x = torch.tensor(np.random.default_rng(2).standard_normal(3 * s.n + n_p), device=DEV)
    x[3 * s.n:] = 0.0
    for call, scalar, bound in ((lambda: s.stokes_qt(x)[0], s.apply, tol), (lambda: s.stokes_operator(x), s.matvec, 1e-13)):
        y = call()
        for c in range(3):
            ref = scalar(x[c * s.n:(c + 1) * s.n].contiguous())
            assert float((y[c * s.n:(c + 1) * s.n] - ref).norm()) <= bound * float(ref.norm())
