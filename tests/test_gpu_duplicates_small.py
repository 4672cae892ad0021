"""Ties at a row's smallest distance, more of them than the perplexity, up to 4,096 points: the
entropy stays above its target at any precision, and the row's affinities go to the tied points in
equal parts. (Above 4,096 points: test_gpu_duplicates.py.)"""
import numpy as np
import pytest
import torch

from paper_1812_09869_amd.tsne import PTSNE, ExactTSNE

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [100, 257, 700, 1024, 1500, 3000, 4096])
@pytest.mark.parametrize("seed", range(4))
def test_more_duplicates_than_the_perplexity(n, seed):
    """40 duplicates at perplexity 20: p = 1 / (39 n) between two of them (each order's 1 / 39,
    halved by 2 n), zero to the others; every row's state finite. FP32 sums of equal numbers and
    two roundings: 1e-6."""
    rng = np.random.Generator(np.random.PCG64(100 * n + seed))
    x = rng.standard_normal((n, 3)) * 10.0 ** rng.uniform(-2, 2)
    dup = rng.choice(n, 40, replace=False)
    x[dup] = 1e4
    print(f"\n[duplicates] n={n} seed={seed}", flush=True)
    model = ExactTSNE(torch.from_numpy(x.astype(np.float32)).cuda(), 20.0)
    beta, _, S, H, _ = (t.cpu().numpy() for t in model.rowstats())
    P = model.p_rows(0, n).cpu().numpy().astype(np.float64)
    assert np.isfinite(beta).all() and np.isfinite(S).all() and np.isfinite(H).all()
    assert np.isfinite(P).all()
    tied = P[np.ix_(dup, dup)]
    off = ~np.eye(40, dtype=bool)
    assert np.abs(tied[off] * 39.0 * n - 1.0).max() <= 1e-6
    others = np.setdiff1d(np.arange(n), dup)
    assert not P[np.ix_(dup, others)].any()
    assert np.abs(S[dup] - 39.0).max() <= 1e-12
    assert model.status() == 0


@pytest.mark.parametrize("n", [100, 257, 1000, 1700, 4000])
def test_tied_dissimilarities(n):
    """Whole-number dissimilarities with zero distances: as above for the rows whose ties exceed
    the perplexity, and every P finite."""
    rng = np.random.Generator(np.random.PCG64(n))
    k = rng.integers(0, 3, n)
    dis = 2.0 * np.abs(k[:, None] - k[None, :])
    print(f"\n[duplicates] dissimilarities n={n}", flush=True)
    model = ExactTSNE.from_dissimilarities(torch.from_numpy(dis.astype(np.float32)).cuda(), 15.0)
    P = model.p_rows(0, n).cpu().numpy().astype(np.float64)
    assert model.status() == 0 and np.isfinite(P).all()
    size = np.bincount(k, minlength=3)
    assert size.min() > 17
    ref = np.where(k[:, None] == k[None, :], 1.0 / (n * (size[k] - 1.0))[:, None], 0.0)
    np.fill_diagonal(ref, 0.0)
    assert np.abs(P - ref).max() <= 1e-6 * ref.max()


@pytest.mark.parametrize("n", [3, 64, 257, 700, 1025, 2048, 3000, 4096, 5000])
def test_identical_points_are_reported(n):
    """All distances of a row equal: no precision to be found, TSNE_E_NONFINITE at every size."""
    print(f"\n[duplicates] identical n={n}", flush=True)
    x = torch.ones(n, 5, device="cuda")
    perp = min(20.0, n / 2.0)
    model = ExactTSNE(x, perp)
    assert model.status() == 5
    assert not torch.isfinite(model.rowstats()[3]).any()
    if n >= 700:  # and as partial problems
        pt = PTSNE(x, 4, 2, perp)
        pt.init_maps(torch.from_numpy(np.random.default_rng(n).standard_normal((n, 2))).float().cuda())
        pt.epoch(torch.arange(n, dtype=torch.int32, device="cuda"))
        assert pt.status() == 5
