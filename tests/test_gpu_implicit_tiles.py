"""Implicit P on both sides of the sizes where its force pass changes: the first whole-tile
problem (9 row blocks), the largest whose triangle the tile buffer holds (63 row blocks, 2,016
tiles) and one past it (65 row blocks, 2,145 tiles, the last block one point; there a workgroup
recomputes and uses tile after tile). Every element's arithmetic and every tile's order of sums
are those of the stored P, so gradient and Z are bitwise equal in every mode; a second pass checks
that nothing of the first one stays."""
import pytest
import torch

from paper_1812_09869_amd import synth
from paper_1812_09869_amd.tsne import ExactTSNE

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["fp64", "fp32", "bf16", "fp16", "bf16x3", "fp16x3"])
@pytest.mark.parametrize("n", [2049, 16128, 16385])
def test_passes_match_stored(n, mode):
    x, lab = synth.gmm_aniso(n, sample_seed=n)
    xt = torch.from_numpy(x).cuda()
    imp = ExactTSNE(xt, 30.0, dist_mode=mode, implicit=True)
    sto = ExactTSNE(xt, 30.0, dist_mode=mode)
    for seed in (9, 10):
        y = torch.from_numpy(synth.clustered_state(lab, seed=seed)).cuda()
        gi, zi = imp.gradient(y, 4.0)
        gs, zs = sto.gradient(y, 4.0)
        assert torch.equal(gi, gs) and torch.equal(zi, zs)
    assert imp.status() == 0 and sto.status() == 0
