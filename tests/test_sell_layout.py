"""The sliced-ELL layout of A_h: its host builder on the CPU, and the
single-vector passes at the sizes where their wavefront split changes."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_layout_decodes_to_the_matrix(tmp_path):
    exe = str(tmp_path / "check")
    host = os.path.join(ROOT, "paper_1204_2586_amd", "csrc", "host")
    subprocess.run(["g++", "-O1", "-std=c++17", "-pthread", os.path.join(ROOT, "tests", "sell_layout_check.cpp"),
                    os.path.join(host, "formats.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip().endswith("OK"), r.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("k,n,index16", [(2, 2, True), (2, 9, True), (3, 5, True), (3, 5, False), (3, 20, True),
                                         (2, 34, True), (2, 34, False), (4, 5, True), (2, 41, True)])
def test_passes_at_every_split(k, n, index16):
    """1, 2, 4 and 8 wavefronts per slice (by the number and length of the
    slices), slices whose length is no multiple of four, 16- and 32-bit
    columns: the product and one application against the host's matrix and a
    handle that is laid out in windows.  The FP64 bound is that of sums of at
    most 400 terms; B of two layouts differs by as much per pass."""
    import torch

    import paper_1204_2586_amd as aux
    import workloads as W
    xyz, tets = W.kuhn_mesh(n, 0.2 if n > 2 else 0.0, 3)
    kw = dict(device="cuda:0", sell_index16=index16)
    a = aux.Solver(xyz, tets, k, sell_window=1 << 30, **kw)
    b = aux.Solver(xyz, tets, k, sell_window=4096, **kw)
    x = torch.tensor(np.random.default_rng(5).standard_normal(a.n), device="cuda:0")
    ref = torch.tensor(a.export_csr("A") @ x.cpu().numpy(), device="cuda:0")
    for s in (a, b):
        assert float((s.matvec(x) - ref).norm() / ref.norm()) <= 400 * 2.0 ** -53
    za, zb = a.apply(x), b.apply(x)
    assert float((za - zb).norm() / za.norm()) <= 1e-12
    for s in (a, b):
        s.set_precision("mixed")
    ya = a.apply(x)
    assert float((ya - za).norm() / za.norm()) <= 2e-6
    assert float((ya - b.apply(x)).norm() / za.norm()) <= 2e-6
