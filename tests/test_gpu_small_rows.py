"""The affinities of many small problems (four rows to a wave up to 1,024
points, one above): partial problems at the edges of a wave's rows, of the
64-point chunks and of the switch, coordinates odd and even in number, against
the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_1812_09869_amd import _lib, synth
from paper_1812_09869_amd.tsne import PTSNE

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("z,d,perp", [(5, 1, 2.0), (31, 2, 5.0), (64, 3, 20.0), (65, 64, 60.0),
                                      (257, 7, 30.0), (1023, 10, 400.0), (1024, 33, 30.0),
                                      (1025, 10, 30.0), (2049, 5, 50.0)])
def test_rows_against_oracle(z, d, perp):
    """Two threads of one layer: problems of z and z - 1 points (n = 2 z - 1).
    beta of every row within 1e-4, P within 1e-5 (Frobenius): the gates of the
    single-problem path."""
    n = 2 * z - 1
    rng = np.random.Generator(np.random.PCG64(100 + n + d))
    x = (rng.standard_normal((n, d)) * rng.uniform(0.1, 30.0)).astype(np.float32)
    print(f"\n[small] z={z} d={d} perplexity={perp}", flush=True)
    model = PTSNE(torch.from_numpy(x).cuda(), 2, 1, perp, iters=1)
    model.init_maps(torch.from_numpy(synth.disk_init(n, 3)))
    order = rng.permutation(n).astype(np.int32)
    model.epoch(torch.from_numpy(order).cuda())
    assert model.status() == 0
    at = 0
    for k in range(2):
        ws, nk = _lib.pt_partial(n, d, model.opts, model.ws, k)
        rows = order[at:at + nk]
        at += nk
        st = oracle.calibrate(x[rows], perp)
        beta = _lib.export_rowstats(ws, nk)[0].cpu().numpy()
        assert np.abs(beta / st.beta - 1.0).max() <= 1e-4
        P = oracle.joint_p(x[rows], st)
        got = _lib.export_p_rows(ws, nk, 0, nk).cpu().numpy().astype(np.float64)
        assert np.linalg.norm(got - P) <= 1e-5 * np.linalg.norm(P)
