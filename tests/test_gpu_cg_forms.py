"""The two forms of a CG iteration (inner products summed by their consumers
and the direction formed inside the product, or separate finishes), on
handles that take one or the other by their size."""
import numpy as np
import pytest
import torch

import oracle
import paper_1204_2586_amd as aux
import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("k,n,aux_space", [(2, 2, 1), (2, 6, 1), (3, 4, 2), (4, 9, 1)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_iterates_match_oracle(k, n, aux_space, precision):
    """Odd and even iteration limits (the direction buffers alternate), with
    and without graph replay, after a switch of the operator and back."""
    xyz, tets = W.kuhn_mesh(n, 0.2 if n > 2 else 0.0, 2)
    s = aux.Solver(xyz, tets, k, device=DEV, precision=precision, operator="matfree", aux_space=aux_space,
                   sell_window=1 << 30)
    ref = oracle.Problem(xyz, tets, k)
    ref = ref.setup_nested() if aux_space == 2 else ref.setup_amg()
    pcg = ref.pcg_nested if aux_space == 2 else ref.pcg
    b = ref.load(W.manufactured_f)
    f = torch.tensor(b, device=DEV)
    s.set_operator("assembled")
    for maxit in (1, 4, 5):
        x = pcg(b, tol=0.0, maxit=maxit, fp32=precision == "mixed")[0]
        u, info = s.solve(f, tol=0.0, maxit=maxit, check=False)
        assert info.iterations == maxit and info.status == aux.ENOTCONV or n == 2
        v = torch.zeros_like(f)
        s.solve_noalloc(f, v, tol=0.0, maxit=maxit, check=False)
        assert torch.equal(u, v)
        assert np.linalg.norm(u.cpu().numpy() - x) <= (1e-10 if precision == "fp64" else 1e-5) * np.linalg.norm(x)
    u, info = s.solve(f, tol=1e-8)
    hist = s.residual_history()
    assert info.converged and len(hist) == info.iterations + 1 and hist[-1] <= 1e-8


def test_breakdown_is_reported_in_both_forms():
    """r.z <= 0 (a negative smoother weight) stops the solve with the last
    iterate whichever kernel sees it first."""
    for n in (4, 34):
        xyz, tets = W.kuhn_mesh(n)
        s = aux.Solver(xyz, tets, 2, device=DEV, smoother_weight=-1.0)
        f = torch.ones(s.n, dtype=torch.float64, device=DEV)
        u, info = s.solve(f, check=False)
        assert info.status == aux.EBREAKDOWN and bool(torch.isfinite(u).all())
