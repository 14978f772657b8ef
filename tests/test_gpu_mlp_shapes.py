"""The predictor's products at the shapes where a kernel or the choice between
kernels can go wrong: batches around the 16-row tiles, widths around the tiles
and the stages of K, and one shape past each line of the dispatch."""
import numpy as np
import pytest
import torch

from paper_2605_20150_amd import predictor as P

pytestmark = pytest.mark.gpu


def say(msg):
    print(msg, flush=True)


def reference(mlp, x, y, ok):
    """Logits, loss and gradients in double precision with the weights the
    products read (bfloat16) and the FP32 biases, and the hidden units (of the
    one hidden layer) whose sign is certain on every row: their pre-activation
    is further from zero than the products' error bound 2^-14 sum |w a|.  A
    unit nearer than that may be cut by the ReLU on one side only."""
    Ws = [w.to(torch.bfloat16).double() for w, _ in mlp.split(mlp.params)]
    bs = [b.double() for _, b in mlp.split(mlp.params)]
    acts = [x.double()]
    for l, (w, b) in enumerate(zip(Ws, bs)):
        z = acts[-1] @ w.T + b
        acts.append(z if l + 1 == len(Ws) else torch.relu(z))
    z = acts[-1]
    count = x.shape[0] * ok.sum()
    loss = ((torch.clamp(z, min=0) - z * y + torch.log1p(torch.exp(-z.abs()))) * ok).sum() / count
    G = (torch.sigmoid(z) - y) * ok / count
    grads = [None] * len(Ws)
    for l in range(len(Ws) - 1, -1, -1):
        grads[l] = (G.T @ acts[l], G.sum(0))
        if l:
            G = (G @ Ws[l]) * (acts[l] > 0)
    S = acts[0].abs() @ Ws[0].abs().T + bs[0].abs()
    sure = ((acts[0] @ Ws[0].T + bs[0]).abs() > 2.0 ** -14 * S).all(0)
    return z, loss, grads, sure


# dims, batch: what they reach
CASES = [
    ([8, 8, 32], 1),               # one chunk of K, one row, tiles mostly past the edge
    ([24, 40, 96], 16),            # K cut inside a chunk; a full 16-row tile
    ([112, 264, 288], 17),         # two row tiles in the direct kernel; K past one 256-deep stage by a chunk
    ([16, 72, 16384], 33),         # direct kernel, 64-row tiles; 64 stages
    ([16, 520, 544], 64),          # input gradient with a cut last stage and a cut column tile
    ([16, 72, 8192], 65),          # 64 x 64 tiles forward, ragged rows
    ([16, 136, 8224], 70),         # 64 x 64 tiles in the weight gradient, ragged every way
    ([16, 136, 65536], 129),       # 128 x 128 tiles forward and in the weight gradient, ragged both ways
    ([16, 16392, 64], 130),        # 128 x 128 tiles in the input gradient, ragged columns
]


@pytest.mark.parametrize("dims,batch", CASES)
def test_products_match_double_precision(dims, batch):
    say(f"case: dims {dims} batch {batch}")
    mlp = P.MLP(dims, seed=91)
    g = torch.Generator(device="cuda").manual_seed(92)
    mlp.params.add_(0.05 * torch.randn(mlp.P, generator=g, device="cuda"))
    mlp.set_weights([w.cpu().numpy() for w, _ in mlp.split(mlp.params)], [b.cpu().numpy() for _, b in mlp.split(mlp.params)])
    x = torch.randn((batch, dims[0]), generator=g, device="cuda")
    n = dims[-1]
    lab = torch.randint(0, 1 << 31, (batch, n // 32), generator=g, device="cuda", dtype=torch.int64).to(torch.int32)
    valid = torch.full((n // 32,), -1, dtype=torch.int32, device="cuda")
    valid[-1] = 0x00FFFFFF
    shift = torch.arange(32, device="cuda", dtype=torch.int32)
    y = ((lab[..., None] >> shift) & 1).reshape(batch, -1).double()
    ok = ((valid[:, None] >> shift) & 1).reshape(1, -1).double()
    z = mlp.forward(x)
    loss = mlp.backward(x, z, lab, valid)
    ref_z, ref_loss, ref_g, sure = reference(mlp, x, y, ok)
    # an FP32 operand enters as two bf16 halves (relative error 2^-17 at most),
    # a layer's sums and the next layers' weights pass it on: 2^-14 of the
    # output's norm covers the two layers with an FP32 sum's own rounding
    rel = float((z.double() - ref_z).norm() / ref_z.norm())
    say(f"logits {rel:.2e} loss {float(loss) - float(ref_loss):.2e}")
    assert rel <= 2.0 ** -14
    assert abs(float(loss) - float(ref_loss)) <= 2.0 ** -14 * abs(float(ref_loss))
    # the weight gradient drops the lo x lo term of its two split operands
    # (2^-18 of a product) besides; a first-layer row is judged where its unit's
    # sign is certain
    say(f"{int((~sure).sum())} of {sure.numel()} units near zero")
    assert (~sure).float().mean() <= 0.05 or sure.numel() < 100
    for l, ((gw, gb), (rw, rb)) in enumerate(zip(mlp.split(mlp.grad), ref_g)):
        for name, a, b in (("W", gw, rw), ("b", gb, rb)):
            if l == 0:
                a, b = a[sure], b[sure]
            rel = float((a.double() - b).norm() / b.norm())
            say(f"layer {l} d{name} {rel:.2e}")
            assert rel <= 1e-4


def test_every_kernel_gives_a_row_the_same_bits():
    """The forward kernels share one accumulation order, so a row's logits do
    not depend on the batch it comes in."""
    dims = [112, 512, 65536]
    mlp = P.MLP(dims, seed=93)
    g = torch.Generator(device="cuda").manual_seed(94)
    x = torch.randn((200, dims[0]), generator=g, device="cuda")
    full = mlp.forward(x).clone()
    for b in (1, 16, 17, 32, 33, 64, 65, 128):
        say(f"case: batch {b} of 200")
        assert torch.equal(mlp.forward(x[:b]), full[:b])


@pytest.mark.parametrize("offset", [1, 2, 3])
def test_logits_need_no_alignment_but_their_elements(offset):
    """The loss reads the caller's logits wherever they lie: the same bits."""
    say(f"case: logits {4 * offset} bytes past a 16-byte boundary")
    mlp = P.MLP([16, 64, 1056], seed=95)
    g = torch.Generator(device="cuda").manual_seed(96)
    x = torch.randn((37, 16), generator=g, device="cuda")
    lab = torch.randint(0, 1 << 31, (37, 33), generator=g, device="cuda", dtype=torch.int64).to(torch.int32)
    valid = torch.full((33,), -1, dtype=torch.int32, device="cuda")
    z = mlp.forward(x)
    want = mlp.backward(x, z, lab, valid).clone(), mlp.grad.clone()
    buf = torch.empty(z.numel() + 4, device="cuda")
    far = buf[offset:offset + z.numel()].view(z.shape)
    assert torch.equal(mlp.forward(x, far), z) and far.data_ptr() % 16 == 4 * offset
    assert torch.equal(mlp.backward(x, far, lab, valid), want[0]) and torch.equal(mlp.grad, want[1])


def one_layer(n_in, n_out, hidden=None):
    return P.MLP([n_in, n_out] if hidden is None else [n_in, hidden, n_out], seed=97)


def test_forward_tiles_give_the_same_bits():
    """64 x 64 tiles (65 rows, 8192 wide), 128 x 128 (1100 rows) and the direct kernel
    (1, 17, 64 rows)."""
    mlp = one_layer(264, 8192)
    x = torch.randn((1100, 264), generator=torch.Generator(device="cuda").manual_seed(98), device="cuda")
    full = mlp.forward(x).clone()
    for b in (1, 17, 64, 65, 200):
        say(f"case: {b} of 1100 rows")
        assert torch.equal(mlp.forward(x[:b]), full[:b])


def test_input_gradient_kernels_give_the_same_bits():
    """The chain kernel (256 rows) and 128 x 128 tiles (16384 rows): the first
    layer's weight gradient where one row counts is that row's input gradient times
    its input.  The other rows' inputs, and so their hidden units, are zero; rows
    and counted outputs are powers of two, so that dL/dz differs by a factor that
    is one."""
    mlp = one_layer(8, 2080, hidden=512)
    g = torch.Generator(device="cuda").manual_seed(99)
    row = torch.randn(8, generator=g, device="cuda")
    bits = torch.randint(0, 1 << 31, (65,), generator=g, device="cuda", dtype=torch.int64).to(torch.int32)
    valid = torch.full((65,), -1, dtype=torch.int32, device="cuda")
    valid[64] = 0
    got = []
    for rows in (256, 16384):
        say(f"case: {rows} rows")
        x = torch.zeros((rows, 8), device="cuda")
        x[3] = row
        lab = torch.zeros((rows, 65), dtype=torch.int32, device="cuda")
        lab[3] = bits
        mlp.backward(x, mlp.forward(x), lab, valid)
        got.append(mlp.split(mlp.grad)[0][0] * rows)
    assert got[0].any() and torch.equal(*got)


@pytest.mark.parametrize("n_out,n_in", [(8192, 512), (2176, 520), (32768, 256)])
def test_weight_gradient_tiles_give_the_same_bits(n_out, n_in):
    """The first rows and columns of a large weight gradient (64 x 64 or 128 x 128
    tiles) and the small one of those alone (32 x 32 tiles): 32 outputs and 64
    inputs of the layer, over 256 rows.  Their logits are the same, as the other
    inputs' weights are zero, and the other outputs do not count."""
    say(f"case: {n_out} x {n_in}")
    g = torch.Generator(device="cuda").manual_seed(102)
    x = torch.randn((256, n_in), generator=g, device="cuda")
    w = torch.randn((32, 64), generator=g, device="cuda") / 8
    lab = torch.randint(0, 1 << 31, (256, 1), generator=g, device="cuda", dtype=torch.int64).to(torch.int32)
    got = []
    for o, i in ((32, 64), (n_out, n_in)):
        mlp = one_layer(i, o)
        W = torch.zeros((o, i), device="cuda")
        W[:32, :64] = w
        mlp.set_weights([W.cpu().numpy()], [torch.zeros(o).numpy()])
        xs = x[:, :i].contiguous()
        z = mlp.forward(xs)
        valid = torch.zeros(o // 32, dtype=torch.int32, device="cuda")
        valid[0] = -1
        labs = torch.zeros((256, o // 32), dtype=torch.int32, device="cuda")
        labs[:, :1] = lab
        mlp.backward(xs, z, labs, valid)
        dw, db = mlp.split(mlp.grad)[0]
        got.append((dw[:32, :64].clone(), db[:32].clone()))
    assert got[0][0].any() and torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


def test_the_halves_of_a_float():
    """An FP32 operand enters the products as bf16 halves hi + lo, rounded by the
    hardware: the same as rounding to nearest even by integers, for ties, both
    sides of them, and every exponent at which the low half is a normal number."""
    rng = np.random.Generator(np.random.PCG64(103))
    exps = np.arange(26, 254, dtype=np.uint32)
    low = np.concatenate([np.arange(0x7F00, 0x8100), [0, 1, 2, 0xFFFF, 0xFFFE], rng.integers(0, 1 << 16, 800)]).astype(np.uint32)
    top = rng.integers(0, 128, (exps.size, low.size)).astype(np.uint32)
    sign = rng.integers(0, 2, top.shape).astype(np.uint32) << 31
    f = (sign | exps[:, None] << 23 | top << 16 | low[None, :]).reshape(-1)
    f = f[: f.size // 8 * 8].view(np.float32)

    def nearest(v):
        u = v.view(np.uint32).astype(np.uint64)
        return ((u + 0x7FFF + (u >> 16 & 1)) & 0xFFFF0000).astype(np.uint32).view(np.float32)

    hi = nearest(f)
    fits = np.isfinite(hi)
    f, hi = f[fits], hi[fits]
    f, hi = f[: f.size // 8 * 8], hi[: f.size // 8 * 8]
    lo = nearest(f - hi)
    W = np.zeros((32, 8), np.float32)
    W[:8, :8] = np.eye(8)
    mlp = one_layer(8, 32)
    mlp.set_weights([W], [np.zeros(32, np.float32)])
    x = torch.tensor(f.reshape(-1, 8), device="cuda")
    say(f"case: {f.size} values")
    for rows in (x[:64], x):
        z = mlp.forward(rows)[:, :8].cpu().numpy()
        assert np.array_equal(z.reshape(-1), (hi + lo)[: z.size])
