"""Footprints of many tiles: the emission and the per-pair gradient sums are cut
into equal pieces of the instances, so a pair of hundreds or thousands of tiles
spans pieces (and, past 1024 tiles a view, is summed across them)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_20150_amd import synth
from paper_2605_20150_amd.raster import Pool, Rasterizer, bins_views, dense_grad

pytestmark = pytest.mark.gpu


def scene(n_small, n_big, seed):
    """Small Gaussians around the origin and wide, faint ones over the whole view."""
    th = synth.dense_scene(n_small + n_big, seed, extent=1.0, logscale_mu=-3.5, logscale_sigma=0.3).astype(np.float64)
    rng = np.random.Generator(np.random.PCG64([seed, 7]))
    big = rng.permutation(n_small + n_big)[:n_big]
    th[big, 3:6] = rng.normal(1.0, 0.1, size=(n_big, 3))
    th[big, 10] = -3.0
    return th


# width, height, small, big: tiles a view and what they reach
CASES = [
    (64, 48, 5, 1),        # 12 tiles: one piece
    (400, 300, 400, 20),   # 475 tiles: pairs begin in one piece and end in another
    (512, 512, 50, 30),    # 1024 tiles: the last grid summed to the pairs' ends
    (528, 512, 50, 30),    # 1056 tiles: the first grid summed across pieces
    (1200, 800, 300, 3),   # 3750 tiles a pair: a piece inside one pair
]


@pytest.mark.parametrize("width,height,n_small,n_big", CASES)
def test_lists_and_gradient_match_the_oracle(width, height, n_small, n_big):
    print(f"case: {width}x{height}, {n_small} small and {n_big} wide Gaussians, two views, FP64", flush=True)
    th = scene(n_small, n_big, 31)
    cams = [synth.look_at(eye, (0, 0, 0), (0, 0, 1), width, height, float(width)) for eye in ((3, 0, 0.5), (0, -3, 0.2))]
    cm = synth.cams_array(cams)
    rng = np.random.Generator(np.random.PCG64(32))
    dimg = rng.normal(size=(2, 3, height, width))
    rast = Rasterizer("cuda")
    pool = Pool.from_dense(torch.tensor(th, device="cuda"), 256)
    proj, bins, fr = rast.forward(pool, cams)
    # the emission, pair by pair: depth order, row-major tiles of each rectangle
    b = {k: v.cpu().numpy().astype(np.int64) for k, v in bins_views(rast, bins).items()}
    rect = proj.rect.view(-1, 2).cpu().numpy().astype(np.int64) & 0xFFFFFFFF
    nt = bins.tiles_x * bins.tiles_y
    want_rec, want_key = [], []
    for r in b["vis_rec"]:
        x0, y0, x1, y1 = rect[r, 0] & 0xFFFF, rect[r, 0] >> 16, rect[r, 1] & 0xFFFF, rect[r, 1] >> 16
        ys, xs = np.mgrid[y0:y1, x0:x1]
        want_key.append((r // proj.n_pidx * nt + ys * bins.tiles_x + xs).reshape(-1))
        want_rec.append(np.full(ys.size, r))
    want_key, want_rec = np.concatenate(want_key), np.concatenate(want_rec)
    assert np.array_equal(b["inst_rec"], want_rec)
    assert np.array_equal(b["inst_e"], np.argsort(want_key, kind="stable"))
    g = rast.backward(pool, cams, proj, bins, fr, torch.tensor(dimg, device="cuda"))
    gd = dense_grad(proj, g, th.shape[0]).cpu().numpy()
    ref = oracle.backward(th, cm, dimg)
    # both sides in double precision: only the order of at most 10^6 terms per
    # sum differs, 10^6 x 1.1e-16 of the sum of their sizes
    rel = np.linalg.norm(gd - ref) / np.linalg.norm(ref)
    print(f"instances {bins.n_inst}, pairs {bins.n_vis}, relative error {rel:.2e}", flush=True)
    assert rel <= 1e-9
    again = rast.backward(pool, cams, proj, bins, fr, torch.tensor(dimg, device="cuda"))
    assert torch.equal(dense_grad(proj, again, th.shape[0]), dense_grad(proj, g, th.shape[0]))
