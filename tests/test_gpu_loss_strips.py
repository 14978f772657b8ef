"""The loss kernels where their strips of rows can go wrong: a strip gives 12, 23,
34 ... output rows, chosen by how many strips the frames make."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_20150_amd.raster import Rasterizer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("views,height,width", [
    (1, 1, 1), (1, 12, 64), (1, 13, 65), (3, 25, 9),        # 12 rows a strip: just full, one row over
    (8, 60, 1900), (8, 61, 1900), (8, 116, 1900),           # FP32 forward: 12 rows (5 strips), 23 (3, 6), 34 (4)
    (8, 36, 1990), (8, 37, 1990),                           # the same edges for the FP64 forward's line
    (2, 1080, 1920),                                        # 56 rows (FP32 forward), 45 (backward)
])
def test_loss_in_strips_of_all_heights(views, height, width):
    """Against the oracle.  FP32: as for any frame, 2e-6 on the loss and 1e-4 on the
    gradient's norm, over the pixels whose sign(x - y) survives the rounding of the
    inputs to FP32 (one of 5M that does not is 4e-4 of that norm).  FP64: rounding of 2^-53 grows by up to 1 / C2 = 1111 (the
    variance of a flat window), a hundred terms: 1e-11 of the largest gradient."""
    print(f"case: loss on {views} views of {width}x{height}", flush=True)
    rng = np.random.default_rng(7 + height)
    x = rng.uniform(0, 1, size=(views, 3, height, width))
    y = np.clip(x + rng.normal(0, 0.2, size=x.shape), 0, 1)
    L, g = oracle.loss(x, y)
    rast = Rasterizer("cuda")
    x32, y32 = x.astype(np.float32), y.astype(np.float32)
    l32, g32 = rast.loss(torch.tensor(x32, device="cuda"), torch.tensor(y32, device="cuda"))
    assert abs(float(l32) - L) < 2e-6
    sure = np.sign(x32 - y32) == np.sign(x - y)
    assert (~sure).sum() <= 3
    assert np.linalg.norm((g32.double().cpu().numpy() - g)[sure]) < 1e-4 * np.linalg.norm(g)
    l64, g64 = rast.loss(torch.tensor(x, device="cuda"), torch.tensor(y, device="cuda"))
    assert abs(float(l64) - L) < 1e-12
    assert np.abs(g64.cpu().numpy() - g).max() < 1e-11 * np.abs(g).max()
