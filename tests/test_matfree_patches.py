"""Patches of the matrix-free operator: the host builder on the CPU, and the
kernels against the assembled operator at the sizes where their shape changes."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_patches_sum_like_the_mesh(tmp_path):
    exe = str(tmp_path / "check")
    host = os.path.join(ROOT, "paper_1204_2586_amd", "csrc", "host")
    subprocess.run(["g++", "-O1", "-std=c++17", "-pthread", os.path.join(ROOT, "tests", "patch_layout_check.cpp"),
                    os.path.join(host, "formats.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip().endswith("OK"), r.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("k,n", [(2, 1), (2, 3), (2, 20), (2, 24), (2, 29), (3, 1), (3, 2), (3, 15), (3, 23), (4, 1),
                                 (4, 2), (4, 9), (4, 18)])
def test_patches_equal_assembled(k, n):
    """One patch with empty places up to more patches than compute units, and
    every patch size of the three orders.  One application differs from the
    assembled operator's by rounding (sums of at most 400 terms per pass, six
    passes: 400 6 2^-53 < 1e-12; FP32 passes are corrected by nothing, so 2e-6
    as for two assembled layouts), three CG steps in FP64 carry it to 1e-10."""
    import numpy as np
    import torch

    import paper_1204_2586_amd as aux
    import workloads as W
    print(f"[patches k={k} n={n}]", flush=True)
    xyz, tets = W.kuhn_mesh(n, 0.2 if n > 2 else 0.0, 3)
    kappa = np.exp(np.random.default_rng(1).standard_normal(tets.shape[0]))
    s = aux.Solver(xyz, tets, k, kappa, device="cuda:0")
    r = torch.tensor(np.random.default_rng(5).standard_normal(s.n), device="cuda:0")

    def both(f):
        out = []
        for op in ("assembled", "matfree"):
            s.set_operator(op)
            out.append(f())
        return float((out[1] - out[0]).norm() / out[0].norm())

    assert both(lambda: s.solve(r, tol=0.0, maxit=3, check=False)[0]) <= 1e-10
    assert both(lambda: s.apply(r)) <= 1e-12
    s.set_precision("mixed")
    assert both(lambda: s.apply(r)) <= 2e-6
