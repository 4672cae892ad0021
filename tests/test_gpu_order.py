"""The locality order of both tree paths (one workgroup per segment up to 4,096
rows, chunks above; more than 128 coordinates take the column kernels): with
one dominant direction every tile must hold 256 points contiguous along it."""
import numpy as np
import pytest
import torch

from paper_1812_09869_amd import _lib
from paper_1812_09869_amd.tsne import ExactTSNE

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [1, 16, 17, 40, 128, 129])
@pytest.mark.parametrize("n", [512, 4096, 8192])
def test_tiles_follow_the_dominant_direction(n, d):
    """n a power of two times 256, so the tiles are the same whichever way a
    segment is sorted. The direction's spread is 1e4 times the others'."""
    rng = np.random.Generator(np.random.PCG64(n + d))
    u = rng.standard_normal(d)
    u /= np.linalg.norm(u)
    s = rng.permutation(n) * (1e4 / n)
    x = (s[:, None] * u + 0.01 * rng.standard_normal((n, d))).astype(np.float32) + 50.0
    # ranks along the direction, of the points as FP32 has them
    rank = np.argsort(np.argsort(x.astype(np.float64) @ u))
    model = ExactTSNE(torch.from_numpy(x).cuda(), 20.0)
    perm = _lib.export_order(model.ws, n)[0].cpu().numpy()
    assert (np.sort(perm) == np.arange(n)).all()
    tiles = np.sort(rank[perm].reshape(-1, 256), axis=1)
    tiles = tiles[np.argsort(tiles[:, 0])]
    # neighbours in rank may swap across a tile's edge (spacing against noise)
    assert np.abs(tiles.reshape(-1) - np.arange(n)).max() <= 2
    assert model.status() == 0
