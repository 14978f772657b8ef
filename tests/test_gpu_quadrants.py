"""The compositing kernels where a tile's four quadrants (or its pixel rows) and
the batches of its list can go wrong: quadrants cut or missed by the image edge,
lists around the batch sizes, pixels that stop in the middle of a group."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_20150_amd import synth
from paper_2605_20150_amd.raster import Pool, Rasterizer, dense_grad

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width,height", [(7, 3), (8, 16), (9, 17), (24, 8), (41, 56)])
@pytest.mark.parametrize("n,logit", [(0, 0.0), (1, 0.0), (31, -2.0), (64, -4.0), (65, -4.0), (129, -4.0), (400, 4.0)])
def test_image_contributors_and_gradient(width, height, n, logit):
    """Every Gaussian covers the whole image (its list is n long in every tile);
    faint ones let the pixels walk all of it, strong ones stop them early.  Both
    sides in double precision: at most n x 256 terms per sum in another order."""
    print(f"case: {width}x{height}, {n} Gaussians, opacity logit {logit}, FP64", flush=True)
    m = max(n, 1)
    th = synth.dense_scene(m, 41, extent=0.3, logscale_mu=-1.0, logscale_sigma=0.3).astype(np.float64)
    th[:, 10] = logit + 0.2 * np.random.Generator(np.random.PCG64(42)).normal(size=m)
    if n == 0:
        th[:, 0:3] += 1e6     # behind the camera or beyond it: empty lists
    cams = [synth.look_at((2.5, 0.3, 0.4), (0, 0, 0), (0, 0, 1), width, height, 0.8 * max(width, height))]
    cm = synth.cams_array(cams)
    dimg = np.random.Generator(np.random.PCG64(43)).normal(size=(1, 3, height, width))
    ref = oracle.render(th, cm)
    rast = Rasterizer("cuda")
    pool = Pool.from_dense(torch.tensor(th, device="cuda"), 256)
    proj, bins, fr = rast.forward(pool, cams)
    assert bins.n_vis == n
    assert np.abs(fr.image.cpu().numpy() - ref["image"]).max() <= 1e-12
    assert np.array_equal(fr.last.cpu().numpy(), ref["last"])
    assert int(fr.visits[0].sum()) == int(ref["visits"].sum())
    assert int(fr.visits[1].sum()) == int(ref["last"].astype(np.int64).sum())
    g = rast.backward(pool, cams, proj, bins, fr, torch.tensor(dimg, device="cuda"))
    gd = dense_grad(proj, g, m).cpu().numpy()
    want = oracle.backward(th, cm, dimg)
    if n == 0:
        assert not gd.any() and not want.any()
    else:
        assert np.linalg.norm(gd - want) <= 1e-10 * np.linalg.norm(want)


@pytest.mark.parametrize("dtype,rtol", [(torch.float32, 2e-4), (torch.float64, 5e-13)])
@pytest.mark.parametrize("n,extent,logscale", [(25, 0.3, -1.5), (400, 0.3, -1.5), (400, 0.02, -5.0)])
def test_backward_of_few_and_of_many_tiles(n, extent, logscale, dtype, rtol):
    """The backward compositing kernels (eight waves a tile in small grids, in short
    batches or, where a few lists are far longer than the others, as in the last
    scene, in long ones; one wave in large grids: over 5120 tiles) form every
    entry's sums by the same operations in the same order: 8 views of 675 tiles,
    one with a dL/dimage and the others without, give that view's gradient.  What differs is the order in which a
    Gaussian's tiles are added (64 at a time in a scan, so at most 6 + 12
    roundings), of terms that may cancel to a hundredth."""
    print(f"case: {n} Gaussians, {extent}, {logscale}, {dtype}", flush=True)
    w, h, m = 425, 391, 8
    th = torch.tensor(synth.dense_scene(n, 44, extent=extent, logscale_mu=logscale, logscale_sigma=0.6), device="cuda",
                      dtype=dtype)
    cams = [synth.look_at((2.5, 0.3, 0.4 + 0.1 * i), (0, 0, 0), (0, 0, 1), w, h, 350.0) for i in range(m)]
    rast = Rasterizer("cuda")
    pool = Pool.from_dense(th, 256)
    dimg = torch.tensor(np.random.Generator(np.random.PCG64(45)).normal(size=(1, 3, h, w)), device="cuda", dtype=dtype)
    got = []
    for views in (1, m):
        d = torch.zeros((views, 3, h, w), device="cuda", dtype=dtype)
        d[0] = dimg[0]
        proj, bins, fr = rast.forward(pool, cams[:views])
        got.append(dense_grad(proj, rast.backward(pool, cams[:views], proj, bins, fr, d), n).cpu())
    assert got[0].abs().max() > 0
    assert (got[0] - got[1]).norm() <= rtol * got[0].norm()
