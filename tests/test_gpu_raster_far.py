"""Rasters at the ends of what the call takes: cells so far out that squared distances overflow
FP32 (every kernel is zero there, and the density is 0), and rasters of very many tiles."""
import math

import pytest
import torch

from paper_1812_09869_amd import _lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 64, 255, 256, 4097])
@pytest.mark.parametrize("x0,y0", [(1e20, 0.0), (0.0, -3e25), (1e20, 1e20)])
def test_cells_beyond_fp32_squares(n, x0, y0):
    gen = torch.Generator(device="cuda").manual_seed(n)
    y = torch.randn(n, 2, generator=gen, device="cuda")
    beta = torch.rand(n, generator=gen, device="cuda", dtype=torch.float64) + 0.5
    out = torch.full((40, 50), -1.0, device="cuda")
    _lib.kde_raster(y, beta, x0, y0, 1.0, 1.0, 50, 40, out)
    assert (out == 0).all()


@pytest.mark.parametrize("along", ["x", "y"])
def test_one_row_of_many_cells(along):
    """One row or column of 2^27 + 100 cells, 2^22 + 4 tiles: more than one launch dimension holds.
    One point of precision 1 whose kernel is flat over a cell: the first cells, the last and those
    about the point within 1e-6 of the peak (FP32 cell centres up to 2^27 / 2^20 = 128)."""
    g = (1 << 27) + 100
    c = 2.0 ** -20
    at = 100.25
    p = (at, 0.5) if along == "x" else (0.5, at)
    y = torch.tensor([p], device="cuda")
    beta = torch.ones(1, dtype=torch.float64, device="cuda")
    out = torch.full((1, g) if along == "x" else (g, 1), -1.0, device="cuda")
    print(f"\n[raster] {g} cells along {along}", flush=True)
    cx, cy, gx, gy = (c, 1.0, g, 1) if along == "x" else (1.0, c, 1, g)
    _lib.kde_raster(y, beta, 0.0, 0.0, cx, cy, gx, gy, out)
    flat = out.view(-1)
    assert float(flat.min()) >= 0.0  # every cell written
    peak = c / math.pi
    k = torch.tensor([0, 1, 31, 32, int(at / c) - (1 << 19), int(at / c), int(at / c) + 5, g - 33,
                      g - 1], device="cuda")
    d = (k.double() + 0.5) * c - at
    ref = peak * torch.exp(-d * d)
    assert float((flat[k].double() - ref).abs().max()) <= 1e-6 * peak + 2.0 * peak * 2.0 ** -17
