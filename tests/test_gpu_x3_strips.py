"""Distances of the x3 modes at the edges of their launch and K loop: 2, 9 and 18 row blocks
(column strips dealt to the eight XCDs, the last turn incomplete), one, two and four steps of 32
coordinates, against the oracle's P. The modes carry about one FP32 rounding of d (2^-23 with the
norms' pair), so a p whose exponent is below 40 moves by 40 * 2^-23 = 5e-6 and the search's
tolerance by 1e-6: relative Frobenius <= 1e-5, the gate of the affinity path; the rows' sums of
the implicit path, recomputed from the same operands, bitwise."""
import numpy as np
import pytest
import torch

import oracle
from paper_1812_09869_amd.tsne import ExactTSNE

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["bf16x3", "fp16x3"])
@pytest.mark.parametrize("n,d", [(300, 20), (2100, 50), (4400, 100)])
def test_x3_distances(n, d, mode):
    rng = np.random.Generator(np.random.PCG64(n + d))
    x = (rng.standard_normal((n, d)) + 8.0 * rng.integers(0, 3, (n, 1))).astype(np.float32)
    st = oracle.calibrate(x, 30.0)
    xt = torch.from_numpy(x).cuda()
    model = ExactTSNE(xt, 30.0, dist_mode=mode)
    beta = model.rowstats()[0].cpu().numpy()
    got = model.p_rows(0, n).cpu().numpy().astype(np.float64)
    P = oracle.joint_p(x, st)
    assert model.status() == 0
    assert np.linalg.norm(got - P) <= 1e-5 * np.linalg.norm(P)
    imp = ExactTSNE(xt, 30.0, dist_mode=mode, implicit=True)
    assert torch.equal(imp.rowstats()[0].cpu(), torch.from_numpy(beta))
