"""Row tiles of the batched products: the host builder on the CPU, and the
kernels against the 64-row slices at the sizes where their shape changes."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_tiles_decode_to_the_matrix(tmp_path):
    exe = str(tmp_path / "check")
    host = os.path.join(ROOT, "paper_1204_2586_amd", "csrc", "host")
    subprocess.run(["g++", "-O1", "-std=c++17", "-pthread", os.path.join(ROOT, "tests", "tile_layout_check.cpp"),
                    os.path.join(host, "formats.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip().endswith("OK"), r.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("k,n,nrhs,order", [(2, 1, 5, 0), (2, 2, 8, 0), (2, 5, 13, 0), (2, 9, 32, 1), (2, 9, 64, 0),
                                            (3, 3, 8, 0), (3, 6, 64, 0), (3, 6, 16, 1), (4, 3, 8, 0), (4, 4, 32, 0),
                                            (4, 4, 64, 0), (2, 21, 32, 0)])
def test_tiles_equal_slices(k, n, nrhs, order):
    """Every block width (8 to 64 columns, so one to four pieces per block row,
    half and whole wavefronts per group), one row to more tiles than
    workgroups, an initial guess (the residual form): three CG steps with tiles
    and with slices.  A row's sum is the same in both; the inner products are
    grouped differently, n 2^-53 relative at worst per product and far less in
    practice, and three steps carry that into U with the condition of the
    preconditioned steps: 1e-10, in mixed precision 1e-5 (the first products'
    differences round to other FP32 numbers: 2^-24 per pass)."""
    import numpy as np
    import torch

    import paper_1204_2586_amd as aux
    import workloads as W
    xyz, tets = W.kuhn_mesh(n, 0.2 if n > 2 else 0.0, 3)
    kw = dict(device="cuda:0", batch_order=order)
    a = aux.Solver(xyz, tets, k, batch_tiles=2, **kw)
    b = aux.Solver(xyz, tets, k, batch_tiles=0, **kw)
    c = aux.Solver(xyz, tets, k, **kw)                   # the fastest: mostly 32 and 64 rows here
    g = np.random.default_rng(7)
    F, U0 = (torch.tensor(g.standard_normal((a.n, nrhs)), device="cuda:0") for _ in range(2))
    for prec, tol in (("fp64", 1e-10), ("mixed", 1e-5)):
        out = []
        for s in (a, b, c):
            s.set_precision(prec)
            u, infos = s.solve_batched(F, tol=0.0, U0=U0, maxit=3, check=False)
            out.append(u)
        print(f"[tiles k={k} n={n} nrhs={nrhs} {prec}] {list(a.info.batch_tile_rows)} "
              f"{list(c.info.batch_tile_rows)}", flush=True)
        assert min(a.info.batch_tile_rows) > 0 and max(b.info.batch_tile_rows) == 0
        for u in (out[0], out[2]):
            assert bool(torch.isfinite(u).all())
            assert float((u - out[1]).norm() / out[1].norm()) <= tol
