"""The force pass of small problems (quarter-tile units): sizes at the edges of
a unit, of a tile and of the rule that selects it, against the oracle, and
batches large enough that several units share a workgroup, bitwise against
separate runs."""
import numpy as np
import pytest
import torch

import oracle
from paper_1812_09869_amd import synth
from paper_1812_09869_amd.tsne import BatchedTSNE, ExactTSNE, Schedule

pytestmark = pytest.mark.gpu


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# 64-row units, 256-row tiles; 2,048 points is the largest problem in units,
# above it every tile is one workgroup of one launch (4,097: 17 row blocks).
# k = 1: every tile holds P; far groups: most tiles are all zero.
@pytest.mark.parametrize("n", [5, 64, 65, 255, 256, 257, 321, 1025, 2048, 2049, 4097])
@pytest.mark.parametrize("far", [False, True], ids=["near", "far"])
def test_unit_edges_against_oracle(n, far):
    """Gradient and one step within the per-step gates (1e-4; the momentum
    1e-3), Z within 1e-6."""
    rng = np.random.Generator(np.random.PCG64(7000 + n))
    k = max(1, min(8, n // 40)) if far else 1
    lab = rng.integers(0, k, n)
    means = rng.standard_normal((k, 6)) * (300.0 if far else 0.0)
    x = (means[lab] + rng.standard_normal((n, 6))).astype(np.float32)
    perp = min(20.0, n / 4.0)
    print(f"\n[units] n={n} far={far}", flush=True)
    P = oracle.joint_p(x, oracle.calibrate(x, perp))
    y = synth.clustered_state(lab, seed=11 + n)
    model = ExactTSNE(_t(x), perp)
    for alpha in (1.0, 12.0):
        g_ref, z_ref = oracle.gradient(P, y.astype(np.float64), alpha)
        g, z = model.gradient(_t(y), alpha)
        g = g.cpu().numpy().astype(np.float64)
        assert np.linalg.norm(g - g_ref) <= 1e-4 * np.linalg.norm(g_ref)
        assert abs(float(z.cpu()[0]) - z_ref) <= 1e-6 * z_ref
    st = model.init_state(_t(y))
    yr, ur, gr = y.astype(np.float64), np.zeros((n, 2)), np.ones((n, 2))
    for t in (300, 301):
        model.step(t, st, Schedule())
        oracle.step(P, yr, ur, gr, oracle.schedule(t))
    assert np.linalg.norm(st[0].cpu().numpy() - yr) <= 1e-4 * np.linalg.norm(yr)
    assert np.linalg.norm(st[1].cpu().numpy() - ur) <= 1e-3 * np.linalg.norm(ur)
    assert model.status() == 0


@pytest.mark.parametrize("whole", [False, True], ids=["units", "mixed"])
@pytest.mark.parametrize("count", [30, 50, 100])
def test_units_sharing_a_workgroup(count, whole):
    """720, 1,200 and 2,400 units (one, two and four to a workgroup), and the
    same with problems outside the rule first, between and last in the table:
    bitwise the state of separate runs."""
    rng = np.random.Generator(np.random.PCG64(91))
    ns = [600 + int(v) for v in rng.integers(0, 100, count)]
    if whole:
        ns[0], ns[count // 2], ns[-1] = 2100, 2049, 4200
    probs = [((rng.standard_normal((n, 4)) * 3).astype(np.float32), 8.0) for n in ns]
    y0s = [synth.embedding_init(n, seed=40 + k) for k, n in enumerate(ns)]
    print(f"\n[units] {count} problems", flush=True)
    batched = BatchedTSNE([(_t(x), p) for x, p in probs])
    batched.init_states([_t(y) for y in y0s])
    batched.run(3)
    assert max(m.status() for m in batched.models) == 0
    for k in (0, 1, count // 2 - 1, count // 2, count // 2 + 1, count - 2, count - 1):
        x, p = probs[k]
        single = ExactTSNE(_t(x), p)
        st = single.init_state(_t(y0s[k]))
        single.run(st, 3)
        for a, b in zip(batched.states[k], st):
            assert torch.equal(a, b), k
