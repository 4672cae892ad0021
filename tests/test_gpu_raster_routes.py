"""The raster at both sides of the lines between its kernels: a thread per four cells for up to 16
points and for more than 2,560 tiles of few cells, else tiles of one (256 points), four (1,024
points, or more than 256 tiles) or sixteen waves. Against FP64 sums at the FP32 cell centres."""
import math

import numpy as np
import pytest
import torch

from paper_1812_09869_amd import _lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,gx,gy", [
    (1, 33, 40), (16, 100, 70), (17, 100, 70), (256, 100, 70), (257, 100, 70), (513, 40, 33),
    (1024, 512, 512), (1025, 512, 512), (1025, 513, 511), (5000, 513, 511),
    (300, 81920, 4), (300, 81952, 4), (300, 81952, 5), (300, 4, 81952), (300, 5, 81952),
    (3000, 1, 90001)])
def test_routes(n, gx, gy):
    """Within 5e-6 of the raster's maximum (two FP32 exponentials of arguments good to 2^-23, and
    FP32 sums over 256 points), at up to 20,000 cells, the last ones among them."""
    rng = np.random.Generator(np.random.PCG64(n + gx))
    y = torch.from_numpy((rng.standard_normal((n, 2)) * 3.0).astype(np.float32)).cuda()
    beta = torch.from_numpy(np.exp(rng.uniform(math.log(1e-2), math.log(1e3), n))).cuda()
    x0, y0, w = -4.0, -3.5, 8.0
    cx, cy = float(np.float32(w / gx)), float(np.float32(w / gy))
    out = torch.full((gy, gx), -1.0, device="cuda")
    print(f"\n[raster] n={n} {gy}x{gx}", flush=True)
    _lib.kde_raster(y, beta, x0, y0, cx, cy, gx, gy, out)
    assert float(out.min()) >= 0.0  # every cell written
    cells = gx * gy
    k = np.unique(np.concatenate([rng.integers(0, cells, 20000), np.arange(max(0, cells - 70), cells)]))
    k = torch.from_numpy(k).cuda()
    u, v = (k % gx).double(), (k // gx).double()
    cu = (x0 + (u + 0.5) * cx).float().double()
    cv = (y0 + (v + 0.5) * cy).float().double()
    ref = torch.zeros_like(cu)
    for j0 in range(0, n, 500):
        p, b = y[j0:j0 + 500].double(), beta[j0:j0 + 500]
        r2 = (cu[:, None] - p[:, 0]) ** 2 + (cv[:, None] - p[:, 1]) ** 2
        ref += (b / math.pi * torch.exp(-b * r2)).sum(1)
    ref *= cx * cy / n
    got = out.view(-1)[k].double()
    assert float((got - ref).abs().max()) <= 5e-6 * max(float(ref.max()), 1e-30)
