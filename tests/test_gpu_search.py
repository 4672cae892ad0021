"""The per-row search at the edges of its variants (4, 8, 16, 32 and 64 points a
lane, a wave to four rows or to one; a workgroup to a row above 4,096 points),
from points and from a dissimilarity matrix, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_1812_09869_amd.tsne import ExactTSNE

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("given", ["points", "dissim"])
@pytest.mark.parametrize("n", [4, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097])
def test_search_edges(n, given):
    """beta of every row within 1e-4 and P within 1e-5 (Frobenius), the gates of
    the affinity path; ties and a far outlier among the points."""
    rng = np.random.Generator(np.random.PCG64(300 + n))
    x = (rng.standard_normal((n, 5)) * 4.0).astype(np.float32)
    x[n // 2] += 60.0
    if n > 100:
        x[1] = x[0]
    perp = min(30.0, n / 2.0)
    print(f"\n[search] n={n} {given}", flush=True)
    if given == "points":
        model = ExactTSNE(torch.from_numpy(x).cuda(), perp, reorder=False)
        st = oracle.calibrate(x, perp)
        P = oracle.joint_p(x, st)
    else:
        xd = x.astype(np.float64)
        dis = np.sqrt(((xd[:, None, :] - xd[None, :, :]) ** 2).sum(axis=2)).astype(np.float32)
        dis = np.triu(dis, 1)
        dis = np.ascontiguousarray(dis + dis.T)
        model = ExactTSNE.from_dissimilarities(torch.from_numpy(dis).cuda(), perp)
        st = oracle.calibrate_dissim(dis, perp)
        P = oracle.joint_p_dissim(dis, st)
    assert model.status() == 0
    beta = model.rowstats()[0].cpu().numpy()
    assert np.abs(beta / st.beta - 1.0).max() <= 1e-4
    got = model.p_rows(0, n).cpu().numpy().astype(np.float64)
    assert np.linalg.norm(got - P) <= 1e-5 * np.linalg.norm(P)
