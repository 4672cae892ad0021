"""Rasters whose cells lie so far out that squared distances overflow FP32: every kernel is zero
there, and the density is 0."""
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
