"""A workspace for a size also serves every smaller one: the sizes that the library
asks for grow with the problem (host only)."""
import numpy as np
import pytest

from paper_2605_20150_amd import _lib as L


def grows(sizes):
    s = np.array(list(sizes), dtype=np.int64)
    assert (s > 0).all()
    return bool((np.diff(s) >= 0).all())


@pytest.mark.parametrize("dtype", [L.TIDE_F32, L.TIDE_F64])
@pytest.mark.parametrize("views,width", [(1, 64), (1, 1), (3, 130), (8, 64), (1, 1920)])
def test_loss(views, width, dtype):
    lib = L.load()
    assert grows(lib.tide_loss_ws_bytes(views, h, width, dtype) for h in range(1, 20000))
    assert grows(lib.tide_loss_ws_bytes(v, 1080, width, dtype) for v in range(1, 100))
    assert grows(lib.tide_loss_ws_bytes(views, 64, w, dtype) for w in range(1, 20000))


@pytest.mark.parametrize("line", [1 << 12, 1 << 15, 1 << 16, 1 << 20, 1 << 22])
def test_binning(line):
    lib = L.load()
    for cap in (0, 1 << 16):
        for v in (1, 4):
            assert grows(lib.tide_bin_sort_ws_bytes(v, n, 19, 25, cap) for n in range(line // v - 300, line // v + 300))
    assert grows(lib.tide_bin_sort_ws_bytes(2, 1000, 19, 25, c) for c in range(line - 300, line + 300))
    assert grows(lib.tide_bin_sort_ws_bytes(1, 1000, x, 64, 1 << 16) for x in range(1, 3000))


@pytest.mark.parametrize("dtype", [L.TIDE_F32, L.TIDE_F64])
@pytest.mark.parametrize("line", [64, 1 << 13, 1 << 17, 1 << 19, 1 << 20, 1 << 24, (1 << 24) + (1 << 19)])
def test_backward(line, dtype):
    lib, bins = L.load(), L.tide_bins()
    bins.n_cams, bins.n_pidx, bins.tiles_x, bins.tiles_y = 2, 1000, 19, 25

    def size(n):
        bins.n_inst = n
        return lib.tide_render_bwd_ws_bytes(bins, dtype)

    assert grows(size(n) for n in range(max(line - 300, 0), line + 300))


def test_predictor():
    lib, mlp = L.load(), L.tide_mlp()
    mlp.n_layers = 2
    mlp.dims[0], mlp.dims[1], mlp.dims[2] = 16, 136, 8224
    assert grows(lib.tide_mlp_ws_bytes(mlp, b) for b in range(1, 600))
