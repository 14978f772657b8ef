"""Sizes at the ends of what the entry points accept."""
import ctypes as C

import pytest
import torch

from paper_2605_20150_amd import _lib as L
from paper_2605_20150_amd import synth
from paper_2605_20150_amd.raster import Pool, Proj, Rasterizer, _stream

pytestmark = pytest.mark.gpu


def room(gigabytes):
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < gigabytes * 1e9:
        pytest.skip(f"needs {gigabytes} GB of device memory")


def wide_pairs(n, side):
    """n pairs that cover a whole grid of side x side tiles each."""
    dev = "cuda"
    return Proj(rec=torch.zeros(12 * n, device=dev), depth=torch.arange(1, n + 1, device=dev, dtype=torch.float32),
                rect=torch.tensor([0, side | side << 16] * n, device=dev, dtype=torch.int32),
                tiles_touched=torch.full((n,), side * side, device=dev, dtype=torch.int32),
                active=torch.ones(n, device=dev, dtype=torch.int32),
                act_idx=torch.arange(n, device=dev, dtype=torch.int32),
                n_active=torch.tensor([n], device=dev, dtype=torch.int32), n_cams=1, n_pidx=n, dtype=L.TIDE_F32)


@pytest.mark.parametrize("n", [255, 256, 300, 4500])
def test_the_instance_count_is_not_cut_to_32_bits(n):
    """Pairs of 2^24 tiles, counted by each of the scans (in one block and in two);
    from 2^32 - 1 instances on the call is refused."""
    print(f"case: {n} pairs x 2^24 tiles, little room", flush=True)
    side = 4096
    proj = wide_pairs(n, side)
    rast = Rasterizer("cuda")
    ws = rast.buf.get("bin_ws", rast.lib.tide_bin_sort_ws_bytes(1, n, side, side, 1 << 16))
    bins = L.tide_bins()
    code = rast.lib.tide_bin_sort(C.byref(proj.c()), side, side, C.c_void_p(ws.data_ptr()), ws.numel(),
                                  C.byref(bins), C.c_void_p(_stream()))
    assert bins.n_inst == n * side * side
    assert code == (L.TIDE_ECAPACITY if n < 256 else L.TIDE_EINVAL)


def test_the_last_instances_below_32_bits():
    """300 pairs of 2^24 tiles and a workspace that holds nearly 2^32 instances, so
    that the last ones are emitted where the 32-bit offsets wrap: refused, and
    whatever the workspace held before (here keys far beyond the grid), nothing is
    written outside of it."""
    print("case: 300 pairs x 2^24 tiles, room for nearly 2^32 instances", flush=True)
    room(150)
    side = 4096
    proj = wide_pairs(300, side)
    rast = Rasterizer("cuda")
    rast.inst_cap = (1 << 32) - (1 << 20)
    rast.buf.get("bin_ws", rast.lib.tide_bin_sort_ws_bytes(1, 300, side, side, rast.inst_cap)).fill_(255)
    with pytest.raises(L.TideError, match="32-bit"):
        rast.bin_sort(proj, side, side)
    torch.cuda.synchronize()
    del rast
    torch.cuda.empty_cache()


def test_an_image_of_more_than_2_to_the_24_tiles():
    """Eight views of 33 x 65535 tiles, one Gaussian near the lower end of each: the
    last rows are those of a small view moved along, the others the background."""
    print("case: 8 views of 513x1048560", flush=True)
    room(110)
    w, h, low, bg = 513, 16 * 65535, 48, (0.25, 0.5, 0.75)
    th = synth.dense_scene(1, 3, extent=0.0, logscale_mu=-1.5, logscale_sigma=0.1)
    pool = Pool.from_dense(torch.tensor(th, device="cuda", dtype=torch.float32), 1)

    def views(height):
        return [synth.look_at((3.0, 0, 0), (0, 0, 0), (0, 0, 1), w, height, 100.0, cx=500.0 - i, cy=height - 20.0)
                for i in range(8)]

    small = Rasterizer("cuda").forward(pool, views(low), bg)[2]
    assert (small.last > 0).any()
    rast = Rasterizer("cuda")
    fr = rast.forward(pool, views(h), bg)[2]
    for name in ("image", "t_final", "last"):
        assert torch.equal(getattr(fr, name)[..., -low:, :], getattr(small, name)), name
    for v in range(8):
        for c in range(3):
            assert bool((fr.image[v, c, :-low] == bg[c]).all())
        assert bool((fr.t_final[v, :-low] == 1).all()) and not bool(fr.last[v, :-low].any())
    assert torch.equal(fr.visits[1], small.visits[1])
    del fr, rast
    torch.cuda.empty_cache()
