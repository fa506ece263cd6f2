"""Level operators and dense cycles of the batched solve against the
single-vector kernels."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,n,nrhs,rows", [(2, 3, 8, 2048), (2, 12, 5, 2048), (2, 12, 16, 0), (2, 30, 32, 2048),
                                           (2, 30, 64, 0), (3, 15, 5, 2048), (3, 15, 33, 0), (4, 6, 16, 2048),
                                           (2, 42, 8, 2048)])
def test_columns_equal_single_solves(k, n, nrhs, rows):
    """Every block width, levels of one slice up to more than the split rule's
    limit, with and without the dense sub-cycle (few and many rows, remainders
    of 16): three CG steps of a block, column by column against the same steps
    of one vector.  Sums in another order: 1e-10, in mixed precision 1e-5 (FP32
    passes round differently, 2^-24 each)."""
    import numpy as np
    import torch

    import paper_1204_2586_amd as aux
    import workloads as W
    print(f"[batch levels k={k} n={n} nrhs={nrhs} rows={rows}]", flush=True)
    xyz, tets = W.kuhn_mesh(n, 0.2 if n > 3 else 0.0, 3)
    s = aux.Solver(xyz, tets, k, device="cuda:0", dense_cycle_rows=rows)
    F = torch.tensor(np.random.default_rng(3).standard_normal((s.n, nrhs)), device="cuda:0")
    for prec, tol in (("fp64", 1e-10), ("mixed", 1e-5)):
        s.set_precision(prec)
        U, _ = s.solve_batched(F, tol=0.0, maxit=3, check=False)
        for j in (0, nrhs // 2, nrhs - 1):
            u, _ = s.solve(F[:, j].contiguous(), tol=0.0, maxit=3, check=False)
            assert float((U[:, j] - u).norm() / u.norm()) <= tol
