"""The tile kernels of the batched products, called one by one on tiles built
here (see Tiles in setup.hpp): every tile size, block width and type, fewer and
more tiles than the 1024 workgroups of a launch, tiles cut short down to one
row, and rows with more columns than a launch requests at once.  A handle
chooses the size by time, so no solve is sure to reach them all."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
LONG = 400                                        # entries of a long row, alone in its tile


class View(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("n", "tile", "ntiles", "max_cols")] + \
               [(n, ctypes.c_void_p) for n in ("rows", "grp_off", "col_off", "ucols", "lidx", "val")]


def _matrix(n, rng):
    """CSR of rows with 1 to 19 entries near the diagonal, and now and then one of LONG."""
    import scipy.sparse as sp
    rows, cols = [], []
    for i in range(n):
        if i % 3000 == 1500:
            c = np.unique((i + rng.integers(-300, 300, 3 * LONG)) % n)[:LONG]
        else:
            c = np.unique(np.append((i + rng.integers(-40, 41, rng.integers(0, 19))) % n, i))
        rows.append(np.full(len(c), i))
        cols.append(c)
    r, c = np.concatenate(rows), np.concatenate(cols)
    return sp.csr_matrix((rng.standard_normal(len(r)), (r, c)), shape=(n, n))


def _tiles(A, tile, rng):
    """The tiles' arrays as numpy, rows in their own order, numbers as they are."""
    n, length = A.shape[0], np.diff(A.indptr)
    first, r = [], 0
    while r < n:
        first.append(r)
        most = tile if rng.random() < 0.9 else int(rng.integers(1, tile + 1))
        end = min(n, r + most)
        long = np.flatnonzero(length[r:end] >= LONG // 2)
        r = r + 1 if len(long) and long[0] == 0 else (r + int(long[0]) if len(long) else end)
    first.append(n)
    nt, groups = len(first) - 1, tile // 8
    rows = np.full(nt * tile, -1, np.int32)
    grp, ucols, lidx, val, col_off = [0], [], [], [], [0]
    for t in range(nt):
        mine = np.arange(first[t], first[t + 1])
        mine = mine[np.argsort(-length[mine], kind="stable")]
        rows[t * tile:t * tile + len(mine)] = mine
        u = np.unique(A.indices[A.indptr[first[t]]:A.indptr[first[t + 1]]])
        ucols.append(u)
        col_off.append(col_off[-1] + len(u))
        for g in range(groups):
            part = mine[8 * g:8 * g + 8]
            blocks = -(-int(length[part[0]]) // 8) if len(part) else 0
            pos, v = np.zeros((blocks, 8, 8), np.uint16), np.zeros((blocks, 8, 8))
            for k, i in enumerate(part):
                e = slice(A.indptr[i], A.indptr[i + 1])
                j = np.arange(length[i])
                p = np.searchsorted(u, A.indices[e])
                pos[:, k, :] = p[-1]
                pos[j // 8, k, j % 8] = p
                v[j // 8, k, j % 8] = A.data[e]
            lidx.append(pos.reshape(-1))
            val.append(v.reshape(-1))
            grp.append(grp[-1] + blocks)
    out = dict(rows=rows, grp_off=np.array(grp, np.int32), col_off=np.array(col_off, np.int32),
               ucols=np.concatenate(ucols).astype(np.int32), lidx=np.concatenate(lidx), val=np.concatenate(val))
    out["max_cols"] = int(np.diff(out["col_off"]).max())
    # the kernels rely on all of this
    assert len(out["lidx"]) == len(out["val"]) == 64 * out["grp_off"][-1] and len(grp) == nt * groups + 1
    assert out["ucols"].min() >= 0 and out["ucols"].max() < n and np.diff(out["col_off"]).min() > 0
    for t in range(nt):
        b = slice(64 * grp[t * groups], 64 * grp[(t + 1) * groups])
        assert out["lidx"][b].max() < col_off[t + 1] - col_off[t]
    assert np.array_equal(np.sort(rows[rows >= 0]), np.arange(n))
    return out


SYMBOL = {"sweep dd": "_ZN4auxp11btile_sweepIdddEEiP12ihipStream_tiRKNS_12DevTilesViewEPKT_PKT0_S8_PT1_PdPKi",
          "sweep ff": "_ZN4auxp11btile_sweepIfffEEiP12ihipStream_tiRKNS_12DevTilesViewEPKT_PKT0_S8_PT1_PdPKi",
          "sweep fd": "_ZN4auxp11btile_sweepIfdfEEiP12ihipStream_tiRKNS_12DevTilesViewEPKT_PKT0_S8_PT1_PdPKi",
          "resid d": "_ZN4auxp11btile_residIdEEiP12ihipStream_tiRKNS_12DevTilesViewEPKT_S8_PS6_PKi",
          "resid f": "_ZN4auxp11btile_residIfEEiP12ihipStream_tiRKNS_12DevTilesViewEPKT_S8_PS6_PKi",
          "spmv64": "_ZN4auxp12btile_spmv64EP12ihipStream_tiRKNS_12DevTilesViewEPKdPdS7_PKi",
          "residual64": "_ZN4auxp16btile_residual64EP12ihipStream_tiRKNS_12DevTilesViewEPKdS6_Pd"}


@pytest.mark.parametrize("many", [False, True])
@pytest.mark.parametrize("tile", [32, 64, 128])
def test_every_tile_size(tile, many):
    """Against scipy in FP64 on the numbers that the kernel is given.  A row's
    sum of m products (and the two operations after it) is within (m + 4) eps of
    the sum of its terms' absolute values in whatever order; an inner product
    of n terms within (n + 4) 2^-53 of theirs."""
    import torch

    import paper_1204_2586_amd as aux
    lib = aux.load_library()
    fn = {k: getattr(lib, s) for k, s in SYMBOL.items()}
    for f in fn.values():
        f.restype = ctypes.c_int
    rng = np.random.default_rng(tile + many)
    n = tile * 1100 + 5 if many else 5 * tile + 3
    A = _matrix(n, rng)
    host = _tiles(A, tile, rng)
    assert (len(host["col_off"]) - 1 > 1024) == many
    dev = {k: torch.tensor(v.astype(np.int16) if k == "lidx" else v, device="cuda:0") for k, v in host.items()
           if k not in ("max_cols", "val")}
    absA = abs(A)
    m = (np.diff(A.indptr) + 4)[:, None]
    p = lambda t: ctypes.c_void_p(t.data_ptr() if t is not None else None)  # noqa: E731
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)

    for width in (8, 16, 32, 64):
        for name in SYMBOL:
            f32 = name.endswith("f") or name == "sweep fd"
            T, eps = (np.float32, 2.0 ** -24) if f32 else (np.float64, 2.0 ** -53)
            val = torch.tensor(host["val"].astype(T), device="cuda:0")
            view = View(n, tile, len(host["col_off"]) - 1, host["max_cols"], *(dev[k].data_ptr() for k in
                        ("rows", "grp_off", "col_off", "ucols", "lidx")), val.data_ptr())
            assert host["max_cols"] * min(128, width * T().itemsize) <= 65536       # the LDS limit of these kernels
            At, absAt = A.astype(T).astype(np.float64), absA.astype(T).astype(np.float64)
            X = rng.standard_normal((n, width)).astype(T)
            F = rng.standard_normal((n, width)).astype(np.float64 if name == "sweep fd" else T)
            d = rng.uniform(0.5, 1.0, n).astype(T)
            x, f, di = (torch.tensor(a, device="cuda:0") for a in (X, F, d))
            y = torch.full_like(x, 7.0)
            parts = torch.zeros(1024 * width, dtype=torch.float64, device="cuda:0")
            print(f"[tile {tile} tiles {view.ntiles} width {width}] {name}", flush=True)
            AX, aAX = At @ X.astype(np.float64), absAt @ np.abs(X.astype(np.float64))
            Fw = F.astype(T).astype(np.float64)
            dot = None
            if name.startswith("sweep"):
                stopped = torch.ones(1, dtype=torch.int32, device="cuda:0")
                fn[name](stream, width, ctypes.byref(view), p(di), p(f), p(x), p(y), None, p(stopped))
                assert bool((y == 7.0).all())
                fn[name](stream, width, ctypes.byref(view), p(di), p(f), p(x), p(y), None, None)
                plain = y.clone()
                g = fn[name](stream, width, ctypes.byref(view), p(di), p(f), p(x), p(y), p(parts), None)
                assert torch.equal(plain, y)
                dd = d.astype(np.float64)[:, None]
                want, size = X + dd * (Fw - AX), np.abs(X) + dd * (np.abs(Fw) + aAX)
                dot = F.astype(np.float64)
            elif name.startswith("resid "):
                fn[name](stream, width, ctypes.byref(view), p(f), p(x), p(y), None)
                want, size = Fw - AX, np.abs(Fw) + aAX
            elif name == "spmv64":
                fn[name](stream, width, ctypes.byref(view), p(x), p(y), None, None)
                plain = y.clone()
                g = fn[name](stream, width, ctypes.byref(view), p(x), p(y), p(parts), None)
                assert torch.equal(plain, y)
                want, size, dot = AX, aAX, X
            else:
                fn[name](stream, width, ctypes.byref(view), p(f), p(x), p(y))
                want, size = Fw - AX, np.abs(Fw) + aAX
            got = y.cpu().numpy().astype(np.float64)
            assert np.all(np.abs(got - want) <= m * eps * size), float((np.abs(got - want) / (m * eps * size)).max())
            if dot is not None:
                sums = parts[:g * width].reshape(g, width).sum(0).cpu().numpy()
                assert np.all(np.abs(sums - (dot * got).sum(0)) <= (n + 4) * 2.0 ** -53 * np.abs(dot * got).sum(0))
