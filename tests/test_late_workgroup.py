"""The stop flag of a CG solve, set in the launch that tests it: on the CPU, the
kernels themselves as a late workgroup runs them (see late_workgroup_check.cpp);
on the GPU, a solve that stops on p.q."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_wavefronts_of_a_late_workgroup_agree(tmp_path):
    tests, exe = os.path.join(ROOT, "tests"), str(tmp_path / "check")
    clang = shutil.which("amdclang++") or os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm/bin/clang++")
    subprocess.run([clang, "-x", "c++", "-std=c++17", "-O1", "-w", "-pthread", "-I", os.path.join(tests, "host_hip"),
                    os.path.join(tests, "late_workgroup_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip() == "OK", r.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("n,weight,operator", [(6, 6.0, "assembled"), (12, 6.0, "assembled"), (36, 8.0, "assembled"),
                                               (6, 6.0, "matfree")])
def test_overflow_of_pq_leaves_the_iterate(n, weight, operator):
    """A large smoother weight makes B indefinite, so a smooth and a rough part
    can be mixed for which p.Ap is 16 times the terms of r.z > 0; scaled so that
    those come to 2^1020 to 2^1022, p.Ap is not finite, and the solve has to end with the
    NaN status before its first update, in both forms of the iteration (n = 36
    has a launch for each sum).  kappa = 2^-300 keeps f.f far from the overflow
    and scales every number exactly."""
    import numpy as np
    import torch

    import paper_1204_2586_amd as aux
    import workloads as W
    xyz, tets = W.kuhn_mesh(n, 0.1, 1)
    s = aux.Solver(xyz, tets, 2, np.full(len(tets), 2.0 ** -300), device="cuda:0", smoother_weight=weight, operator=operator)
    rough = s.matvec(torch.tensor(np.random.default_rng(0).standard_normal(s.n), device="cuda:0"))
    smooth = s.matvec(torch.tensor(np.prod(np.sin(np.pi * xyz[s.dof_keys()].mean(1)), 1), device="cuda:0"))

    def form(a, b):
        return float(a @ s.apply(b))
    c0, c1, c2 = form(smooth, smooth), form(smooth, rough) + form(rough, smooth), form(rough, rough)
    assert c0 > 0 > c2
    r = smooth + max(np.roots([c2, c1, 0.5 * c0]).real) * rough       # r.z = c0 / 2
    z = s.apply(r)
    terms, pq = float((r * z).abs().sum()), float(z @ s.matvec(z))
    print(f"[pq n={n} {operator}] {pq / terms:.3g} times", flush=True)
    assert float(r @ z) > 0 and pq > 2 ** 4 * terms
    f = r * 2.0 ** np.floor(0.5 * (1022 - np.log2(terms)))
    assert bool(torch.isfinite(f @ f))
    u, info = s.solve(f, check=False)
    assert info.status == aux.ENAN and info.iterations == 0
    assert torch.equal(u, torch.zeros_like(f))
