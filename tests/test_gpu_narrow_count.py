"""aux_info counts the slices that store 16-bit columns, in one range or two."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime, before the library's)

import paper_1204_2586_amd as aux
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,window", [(24, 1 << 30), (24, 4096), (40, 1 << 30)])
def test_count_agrees_with_the_column_bytes(n, window):
    """A stored entry takes 4 bytes of columns in a 32-bit slice and 2 + 8 / 64
    in a 16-bit one, so the bytes tell how many entries the 32-bit slices hold:
    between the shortest and the longest row, in groups of four, for each."""
    xyz, tets = W.kuhn_mesh(n, 0.2, 1)
    s = aux.Solver(xyz, tets, 2, device="cuda:0", sell_window=window)
    i = s.info
    length = np.diff(s.export_csr("A").indptr)
    wide = (i.sell_index_bytes - 2.125 * i.stored_A) / 1.875
    slices = i.sell_slices - i.sell_narrow_slices
    print(f"[narrow n={n}] {i.sell_narrow_slices} of {i.sell_slices}, {wide:.0f} entries in the others", flush=True)
    assert slices * 64 * 4 * -(-length.min() // 4) <= wide <= slices * 64 * 4 * -(-length.max() // 4)
