"""Passes of the row search where far points make up a row's variance: the search starts from the
variance, so its first bracket is many orders of magnitude wide."""
import numpy as np
import pytest
import torch

import oracle
from paper_1812_09869_amd.tsne import ExactTSNE

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [150, 700, 1500, 4000])
@pytest.mark.parametrize("kind", ["two", "ten", "stray"])
def test_far_points_and_passes(n, kind):
    """At most 14 passes for any row: the bracket is at most 2^53 wide (distances in FP32, squared
    spread over width 1e8), so six halvings of its exponent leave less than a factor of two, and
    Newton's steps with the two of the start take eight. Precisions are the oracle's (1e-4)."""
    rng = np.random.Generator(np.random.PCG64(n))
    x = rng.standard_normal((n, 6))
    if kind == "stray":
        x[n // 3] += 1e4
    else:
        x += 1e3 * rng.integers(0, 2 if kind == "two" else 10, (n, 1))
    x = x.astype(np.float32)
    for perp in (5.0, 30.0):
        model = ExactTSNE(torch.from_numpy(x).cuda(), perp)
        assert model.status() == 0
        beta, _, _, _, evals = (t.cpu().numpy() for t in model.rowstats())
        rows = rng.choice(n, 40, replace=False)
        ref = oracle.calibrate(x, perp, rows=rows).beta
        print(f"\n[start] n={n} {kind} perplexity {perp:g}: passes {evals.mean():.1f}, at most "
              f"{evals.max()}", flush=True)
        assert np.abs(beta[rows] / ref - 1.0).max() <= 1e-4
        assert evals.min() >= 1 and evals.max() <= 14
