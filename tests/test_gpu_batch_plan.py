"""A batched step whose problem list is not the planned one changes nothing, also where the two
lists have as many problems, row blocks and tiles and differ in the quarter-tile units alone."""
import numpy as np
import pytest
import torch

from paper_1812_09869_amd import _lib, synth
from paper_1812_09869_amd.tsne import BatchedTSNE

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("planned,stepped", [((4, 5, 9), (3, 7, 8)), ((3, 7, 8), (4, 5, 9))])
def test_mismatch_of_units_alone(planned, stepped):
    """Row blocks of the problems: 18 and 70 tiles in both lists, one list with a problem past the
    eight blocks of the units' rule."""
    rng = np.random.Generator(np.random.PCG64(61))
    models = {}
    for name, blocks in (("planned", planned), ("stepped", stepped)):
        ns = [256 * b - 3 for b in blocks]
        xs = [torch.from_numpy(rng.standard_normal((n, 3)).astype(np.float32)).cuda() for n in ns]
        b = BatchedTSNE([(x, 8.0) for x in xs])
        b.init_states([torch.from_numpy(synth.embedding_init(n, seed=n)).cuda() for n in ns])
        models[name] = b
    print(f"\n[plan] {planned} stepped as {stepped}", flush=True)
    states = [t for b in models.values() for st in b.states for t in st]
    before = [t.clone() for t in states]
    cost = torch.full((3, 2), -1.0, dtype=torch.float64, device="cuda")
    _lib.batch_step(models["stepped"]._arr, models["planned"]._bws, 1.0, 0.5, 200.0)
    _lib.batch_cost(models["stepped"]._arr, models["planned"]._bws, cost)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(states, before))
    assert (cost == -1.0).all()
    # the list that was planned still steps
    models["planned"].run(1)
    assert not torch.equal(models["planned"].states[0][0], before[0])
