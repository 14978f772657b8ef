"""The (N, 59) table to block-SoA slots and the compact gradient back to (N, 59), by
one kernel each, against the general torch path: whole values, so equal bits."""
import pytest
import torch

from paper_2605_20150_amd import synth
from paper_2605_20150_amd.raster import D, Pool, Rasterizer, dense_grad

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("n,block_rows,extra", [(1, 1, 0), (63, 64, 1), (64, 64, 0), (65, 64, 2), (1000, 7, 3),
                                                (5000, 4096, 1)])
def test_rows_to_blocks(n, block_rows, extra, dtype):
    print(f"case: {n} rows, blocks of {block_rows}, {extra} spare slots, {dtype}", flush=True)
    theta = torch.randn(n, D, generator=torch.Generator().manual_seed(n), dtype=torch.float64).to(dtype)
    want = Pool.from_dense(theta, block_rows, extra)
    wide = torch.zeros(n, D + 1, dtype=dtype)
    wide[:, :D] = theta
    for th in (theta.cuda(), wide.cuda()[:, :D], theta.cuda().requires_grad_(True)):
        got = Pool.from_dense(th, block_rows, extra)
        assert got.params.requires_grad == th.requires_grad
        for k in ("params", "exp_avg", "exp_avg_sq", "step", "slot_block", "slot_rows", "order"):
            a, b = getattr(got, k).detach().cpu(), getattr(want, k)
            assert a.dtype == b.dtype and torch.equal(a, b), k
        assert (got.n_slots, got.block_rows, got.n_order) == (want.n_slots, want.block_rows, want.n_order)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 700])
def test_dense_gradient(n, dtype):
    print(f"case: {n} rows, {dtype}", flush=True)
    theta = torch.tensor(synth.dense_scene(n, 5), device="cuda", dtype=dtype)
    theta[::3, 0:3] += 1e6          # out of view: rows without a gradient
    cams = [synth.look_at((2.5, 0.3, 0.4), (0, 0, 0), (0, 0, 1), 70, 41, 60.0)]
    rast = Rasterizer("cuda")
    pool = Pool.from_dense(theta, 256)
    proj, bins, fr = rast.forward(pool, cams)
    g = rast.backward(pool, cams, proj, bins, fr, torch.ones_like(fr.image))
    other_stride = g.T.contiguous().T        # takes the general path
    for rows in (1, n // 2 + 1, n):
        got = dense_grad(proj, g, rows)
        assert got.is_contiguous() and torch.equal(got, dense_grad(proj, other_stride, rows))
    # recorded by autograd: the general path, differentiable
    gr = g.clone().requires_grad_(True)
    assert dense_grad(proj, gr, n).requires_grad


def test_traced_programs_see_the_operations():
    """A program recorded on one table runs on another: by jit.trace and by make_fx,
    both of which hand over tensors of values."""
    from torch.fx.experimental.proxy_tensor import make_fx
    a, b = (torch.randn(10, D, generator=torch.Generator().manual_seed(s)).cuda() for s in (1, 2))
    want = Pool.from_dense(b, 4).params
    for record in (lambda f, x: torch.jit.trace(f, x, check_trace=False), lambda f, x: make_fx(f)(x)):
        print("case: a recorded program", flush=True)
        assert torch.equal(record(lambda t: Pool.from_dense(t, 4).params, a)(b), want)
