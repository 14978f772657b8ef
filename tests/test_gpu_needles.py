"""Long thin oblique footprints in single precision: the terms of an entry's power
cancel there, so the tests that pass over whole boxes of pixels have to allow for
the rounding of what they leave out, and both directions have to take exactly the
entries that the per-pixel test takes."""
import math

import numpy as np
import pytest
import torch

from paper_2605_20150_amd.raster import Pool, Rasterizer, dense_grad

pytestmark = pytest.mark.gpu

LOG2E = 1.4426950408889634
C0 = 0.5 * math.sqrt(1.0 / math.pi)


def needles(n, length, width, height, seed):
    """A camera of 100 px a unit at depth 10 and n needles around there, 3 sigma =
    length px and 0.05 to 0.35 px, at all angles, each at a depth of its own."""
    from paper_2605_20150_amd import synth
    cam = synth.look_at((0, 0, 0), (0, 0, 1), (0, -1, 0), width, height, 1000.0)
    rng = np.random.Generator(np.random.PCG64(seed))
    R = np.array(cam.R, dtype=np.float64).reshape(3, 3)
    th = np.zeros((n, 59))
    ang = rng.uniform(0, math.pi, n)
    along = rng.uniform(-0.8, 0.8, n) * length / 100
    p = np.stack([rng.uniform(-1, 1, n) * width / 300 + along * np.cos(ang),
                  rng.uniform(-1, 1, n) * height / 300 + along * np.sin(ang),
                  10 + 0.001 * rng.permutation(n)], 1)
    th[:, 0:3] = (p - np.array(cam.t)) @ R     # camera to world
    sig = np.stack([length / 300 * rng.uniform(0.7, 1.2, n), rng.uniform(0.0005, 0.0035, n)], 1)
    th[:, 3:6] = np.log(sig[:, [0, 1, 1]])
    # the long axis at the angle in the image plane: world axes = R^T camera axes
    for i in range(n):
        c, s = math.cos(ang[i]), math.sin(ang[i])
        th[i, 6:10] = quaternion(R.T @ np.array([[c, -s, 0], [s, c, 0], [0, 0, 1]]))
    th[:, 10] = rng.uniform(-3, 0, n)
    th[:, 11:14] = 0.5
    return th, [cam]


def quaternion(M):
    w, v = np.linalg.eig(M)
    axis = np.real(v[:, np.argmin(abs(w - 1))])
    c = (np.trace(M) - 1) / 2
    s = axis @ np.array([M[2, 1] - M[1, 2], M[0, 2] - M[2, 0], M[1, 0] - M[0, 1]]) / 2
    t = math.atan2(s, c)
    return np.concatenate([[math.cos(t / 2)], math.sin(t / 2) * axis])


def fma(a, b, c):
    """float32 a b + c, rounded once but for double rounding."""
    return (a.double() * b.double() + c.double()).float()


@pytest.mark.parametrize("length", [1000, 3000])
@pytest.mark.parametrize("width,height", [(1024, 512), (2048, 1024)])   # the backward of few and of many tiles
def test_both_directions_take_what_the_pixels_take(width, height, length):
    """The oracle of the decisions is the per-pixel test alone, in float32 on the
    kernels' own records, walked pixel by pixel in depth order.  A lost entry is
    a factor 254/255 of the transmittance.  dL/dimage is nonzero only where some
    entry's alpha lies within 2 % of 1/255, so that a colour gradient is a sum of
    few terms and a lost one is 0.0039 C0 of it.  Bounds: a few hundred factors
    of relative rounding 2^-23 in T (1e-4 of it), and as much of the sum of the
    terms' sizes; pixels with an alpha within 1e-5 of 1/255, which an exponential
    off by an ulp decides, are left out of both."""
    n = 400
    print(f"case: {n} needles of {length} px, {width}x{height}, FP32", flush=True)
    th, cams = needles(n, length, width, height, 61)
    rast = Rasterizer("cuda")
    pool = Pool.from_dense(torch.tensor(th, device="cuda", dtype=torch.float32), 512)
    proj, bins, fr = rast.forward(pool, cams)
    rec = proj.rec.view(-1, 12)[:n].clone()
    rect = proj.rect.view(-1, 2)[:n].cpu().numpy().astype(np.int64) & 0xFFFFFFFF
    seen = proj.tiles_touched[:n].cpu().numpy() > 0
    order = np.argsort(proj.depth[:n].cpu().numpy(), kind="stable")
    k = torch.tensor(LOG2E, device="cuda", dtype=torch.float32)
    px = torch.arange(width, device="cuda", dtype=torch.float32) + 0.5
    py = torch.arange(height, device="cuda", dtype=torch.float32) + 0.5
    T = torch.ones((height, width), device="cuda", dtype=torch.float64)
    unsure = torch.zeros((height, width), device="cuda", dtype=torch.bool)
    edge = torch.zeros_like(unsure)
    gone = torch.zeros_like(unsure)
    walk = []
    for i in order[seen[order]]:
        x0, y0, x1, y1 = rect[i, 0] & 0xFFFF, rect[i, 0] >> 16, rect[i, 1] & 0xFFFF, rect[i, 1] >> 16
        box = np.s_[16 * y0:min(16 * y1, height), 16 * x0:min(16 * x1, width)]
        u, v, A, B, C, op = rec[i, :6]
        dx = (px[box[1]] - u)[None, :]
        dy = (py[box[0]] - v)[:, None]
        power = fma(dy, fma(-0.5 * k * C, dy, -k * B * dx), -0.5 * k * A * dx * dx)
        araw = op * torch.exp2(power)
        unsure[box] |= (power <= 0) & ((araw * 255 - 1).abs() < 1e-5)
        edge[box] |= (power <= 0) & (araw * 255 >= 1) & (araw * 255 < 1.02)
        take = (power <= 0) & (araw >= 1 / 255) & ~gone[box]
        alpha = torch.clamp(araw, max=0.99).double()
        tn = T[box] * (1 - alpha)
        unsure[box] |= take & ((tn / 1e-4 - 1).abs() < 1e-3)
        gone[box] |= take & (tn < 1e-4)
        take &= ~gone[box]
        walk.append((i, box, take, alpha * take * T[box]))
        T[box] = torch.where(take, tn, T[box])
    ok = ~unsure
    rel = ((fr.t_final[0].double() / T - 1).abs() * ok).max()
    print(f"{int(edge.sum())} pixels at an entry's edge, {int(unsure.sum())} left out, T off by {float(rel):.1e}", flush=True)
    assert ok.double().mean() > 0.99 and edge.sum() > 1000
    assert rel <= 1e-4
    d = torch.tensor(np.random.Generator(np.random.PCG64(62)).choice([-1.0, 1.0], size=(height, width)), device="cuda")
    d = d * (edge & ok)
    dimg = torch.zeros_like(fr.image)
    dimg[0, 0] = d.float()
    g = dense_grad(proj, rast.backward(pool, cams, proj, bins, fr, dimg), n).double().cpu().numpy()
    worst = 0.0
    for i, box, take, w in walk:
        want, size = C0 * float((w * d[box]).sum()), C0 * float((w * d[box].abs()).sum())
        worst = max(worst, abs(g[i, 11] - want) / (1e-4 * size + 1e-4))
    print(f"colour gradients off by {worst:.2f} of the bound", flush=True)
    assert worst <= 1
