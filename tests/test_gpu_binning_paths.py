"""The binning where its small-scene paths end: scans that read their predecessors'
elements (to 8 blocks of 4096), depth sorts in tiles of 1024 keys (to 65536 pairs)
and 2048 (to 1048576), tile sorts that add the counts up themselves (to
512 tiles of 4096 by the workspace) and launch orders without a counting launch
(to 4 blocks of 256 tiles).  Every list is a whole number: equal, not close."""
import pytest
import torch

from paper_2605_20150_amd import synth
from paper_2605_20150_amd.raster import Pool, Rasterizer, bins_views

pytestmark = pytest.mark.gpu


def check(rast, proj, bins, tx, ty):
    V, N, T = proj.n_cams, proj.n_pidx, tx * ty
    torch.cuda.synchronize()
    act = (proj.active.long() != 0).long()
    assert torch.equal(proj.act_idx.long()[act > 0], (act.cumsum(0) - act)[act > 0])
    assert int(proj.n_active) == int(act.sum())
    tt = proj.tiles_touched.long()
    vis = tt.nonzero().flatten()
    v = bins_views(rast, bins)
    assert bins.n_vis == vis.numel() and bins.n_inst == int(tt.sum())
    vis = vis[torch.sort(proj.depth.view(torch.int32)[vis], stable=True).indices]   # depths are positive
    assert torch.equal(v["vis_rec"].long(), vis)
    off = torch.zeros(vis.numel() + 1, dtype=torch.long, device=vis.device)
    off[1:] = tt[vis].cumsum(0)
    assert torch.equal(v["inst_off"].long(), off)
    rect = proj.rect.view(-1, 2)[vis].long() & 0xffffffff
    x0, y0, x1 = rect[:, 0] & 0xffff, rect[:, 0] >> 16, rect[:, 1] & 0xffff
    pair = torch.repeat_interleave(torch.arange(vis.numel(), device=vis.device), tt[vis])
    k = torch.arange(pair.numel(), device=vis.device) - off[pair]
    wd = (x1 - x0)[pair]
    tile = vis[pair] // N * T + (y0[pair] + k // wd) * tx + x0[pair] + k % wd
    assert torch.equal(v["inst_rec"].long(), vis[pair])
    key, order = torch.sort(tile, stable=True)
    assert torch.equal(v["inst_e"].long(), order)
    cnt = torch.bincount(key, minlength=V * T)
    rg = v["ranges"].long()
    assert torch.equal(rg[:, 1] - rg[:, 0], cnt)
    assert torch.equal(rg[:, 0][cnt > 0], (cnt.cumsum(0) - cnt)[cnt > 0])
    to = v["tile_order"].long()
    assert torch.equal(torch.sort(to).values, torch.arange(V * T, device=to.device))
    assert cnt[to[0]] >= 0.8 * cnt.max()           # longest first, by length classes


@pytest.mark.parametrize("inst_cap", [1 << 17, 1 << 22])
@pytest.mark.parametrize("n,views,width,height", [
    (1, 1, 16, 16), (500, 1, 64, 64), (4096, 1, 250, 256), (4097, 1, 257, 256),      # one block, two
    (32768, 1, 300, 200), (32769, 1, 300, 200), (9000, 4, 512, 512),                 # eight blocks, nine, twelve
    (16384, 4, 200, 200), (20480, 4, 200, 200),                                      # 65536 pairs at most, 81920
    (262144, 4, 100, 100), (266240, 4, 100, 100),                                    # 1048576, 1064960
    (3000, 1, 512, 512), (3000, 1, 513, 512), (3000, 1, 1040, 1072)])                # 1024 tiles, 1056, 4355
def test_lists(n, views, width, height, inst_cap):
    print(f"case: {n} Gaussians, {views} x {width}x{height}, room for {inst_cap}", flush=True)
    theta = torch.tensor(synth.dense_scene(n, 9, extent=1.0, logscale_mu=-4.0, logscale_sigma=0.5), device="cuda",
                         dtype=torch.float32)
    cams = [synth.look_at((2.5, 0.3, 0.4 + 0.2 * i), (0, 0, 0), (0, 0, 1), width, height, 0.8 * max(width, height))
            for i in range(views)]
    rast = Rasterizer("cuda")
    rast.inst_cap = inst_cap
    proj, bins, _ = rast.forward(Pool.from_dense(theta, 4096 if n > 1 else 1), cams)
    check(rast, proj, bins, -(-width // 16), -(-height // 16))
