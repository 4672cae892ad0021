"""The searches that pass points over: rows in the locality order, whose far points (and, in the
pack, whole tiles) are left alone, and the bandwidths of a map, whose passes read only the points
near enough. Both leave out exact zeros only, so the gates are those of the affinity path (beta
1e-4, P 1e-5 Frobenius)."""
import numpy as np
import pytest
import torch

import oracle
from paper_1812_09869_amd import _lib
from paper_1812_09869_amd.tsne import ExactTSNE

pytestmark = pytest.mark.gpu

FLT_MIN = 2.0 ** -126


@pytest.mark.parametrize("n,apart", [(4097, 3.0), (4352, 300.0), (8193, 20.0)])
def test_zero_tiles(n, apart):
    """A tile's flag is set exactly where the oracle's P holds a normal FP32 number (1% about the
    limit left open: exponents of 87 in FP32), and what is not stored reads as zero."""
    rng = np.random.Generator(np.random.PCG64(n))
    x = (rng.standard_normal((n, 6)) * rng.choice([0.2, 1.0, 3.0], (n, 1))).astype(np.float32)
    x += (apart * rng.integers(0, 5, (n, 1))).astype(np.float32)
    model = ExactTSNE(torch.from_numpy(x).cuda(), 30.0)
    st = oracle.calibrate(x, 30.0)
    beta = model.rowstats()[0].cpu().numpy()
    perm, flags = (t.cpu().numpy() for t in _lib.export_order(model.ws, n))
    assert model.status() == 0
    assert np.abs(beta / st.beta - 1.0).max() <= 1e-4
    P = oracle.joint_p(x, st)
    got = model.p_rows(0, n).cpu().numpy().astype(np.float64)
    assert np.linalg.norm(got - P) <= 1e-5 * np.linalg.norm(P)
    assert not got[P < 0.99 * FLT_MIN].any()
    Q = P[perm][:, perm]
    nb = (n + 255) // 256
    t = 0
    for i in range(nb):
        for j in range(i, nb):
            top = Q[256 * i:256 * (i + 1), 256 * j:256 * (j + 1)].max()
            if top > 1.01 * FLT_MIN:
                assert flags[t] == 1, (i, j, top)
            if top < 0.99 * FLT_MIN:
                assert flags[t] == 0, (i, j, top)
            t += 1


@pytest.mark.parametrize("n", [5, 1024, 1025, 8192, 8193, 20000, 33000])
def test_map_bandwidths(n):
    """Points a lane: 1, 2, 8, 16 (from where they are kept), 32 and 64; clusters of very
    different density, so that a row starts from a precision far above or below its own, ties, a
    far outlier; a map that starts at an odd float."""
    rng = np.random.Generator(np.random.PCG64(n))
    y = rng.standard_normal((n, 2)) * rng.choice([0.01, 1.0, 30.0], (n, 1))
    y += 50.0 * rng.integers(0, 4, (n, 2))
    y[n // 2] += 4000.0
    y[1] = y[0]
    y = y.astype(np.float32)
    perp = min(50.0, n / 2.0)
    flat = torch.zeros(2 * n + 1, device="cuda")
    yt = flat[1:].view(n, 2)
    yt.copy_(torch.from_numpy(y))
    beta = torch.empty(n, dtype=torch.float64, device="cuda")
    _lib.kde_bandwidths(yt, perp, _lib.kde_new_workspace(n), beta)
    rows = np.unique(np.concatenate([rng.integers(0, n, 200), [0, 1, n // 2, n - 1]]))
    ref = oracle.calibrate(y.astype(np.float64), perp, rows=rows).beta
    assert np.abs(beta.cpu().numpy()[rows] / ref - 1.0).max() <= 1e-4
