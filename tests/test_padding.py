"""Padding of the device layouts: a row multiplies no vector entry but those of
its own columns, so an Inf or NaN reaches only the rows that have it."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_padding_stays_in_its_row(tmp_path):
    exe = str(tmp_path / "check")
    host = os.path.join(ROOT, "paper_1204_2586_amd", "csrc", "host")
    subprocess.run(["g++", "-O1", "-std=c++17", "-pthread", os.path.join(ROOT, "tests", "padding_check.cpp"),
                    os.path.join(host, "formats.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "OK", r.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("k,n,index16", [(2, 4, True), (2, 4, False), (2, 9, True), (3, 5, True), (3, 5, False),
                                         (4, 4, True), (2, 26, True)])
def test_infinity_reaches_only_coupled_rows(k, n, index16):
    import torch

    import paper_1204_2586_amd as aux
    import workloads as W
    xyz, tets = W.kuhn_mesh(n, 0.2, 3)
    s = aux.Solver(xyz, tets, k, device="cuda:0", sell_index16=index16)
    A = s.export_csr("A").tocsc()
    g = np.random.default_rng(1)
    x = g.standard_normal(s.n)
    # the longest rows come first in the layout, the shortest last
    length = np.diff(A.tocsr().indptr)
    dofs = {int(length.argmax()), int(length.argmin()), 0, s.n - 1, *map(int, g.integers(0, s.n, 12))}
    for d in dofs:
        for bad in (np.inf, np.nan):
            v = x.copy()
            v[d] = bad
            finite = torch.isfinite(s.matvec(torch.tensor(v, device="cuda:0"))).cpu().numpy()
            want = np.ones(s.n, dtype=bool)
            want[A.indices[A.indptr[d]:A.indptr[d + 1]]] = False
            assert np.array_equal(finite, want), (d, bad, int((finite != want).sum()))
