"""Quarter-tile units of very many problems: more than 16,384, from where a workgroup takes three
steps to find its problem in the table."""
import numpy as np
import pytest
import torch

from paper_1812_09869_amd import synth
from paper_1812_09869_amd.tsne import BatchedTSNE, ExactTSNE

pytestmark = pytest.mark.gpu


def test_more_than_16384_problems():
    """16,500 problems of 4 to 300 points; sampled ones, at the steps' edges among them, are
    bitwise the state of separate runs."""
    count = 16500
    rng = np.random.Generator(np.random.PCG64(71))
    ns = rng.integers(4, 9, count)
    ns[rng.integers(0, count, 40)] = 300  # two row blocks: the units are not a multiple of the index
    xs = [torch.from_numpy((3.0 * rng.standard_normal((int(n), 2))).astype(np.float32)).cuda()
          for n in ns]
    y0s = [torch.from_numpy(synth.embedding_init(int(n), seed=k)).cuda() for k, n in enumerate(ns)]
    print(f"\n[units] {count} problems", flush=True)
    batched = BatchedTSNE([(x, 2.0) for x in xs])
    batched.init_states(y0s)
    batched.run(2)
    edges = [0, 1, 127, 128, 129, 16383, 16384, 16385, count - 2, count - 1]
    for k in sorted({*edges, *(int(v) for v in rng.integers(0, count, 40)),
                     *(int(v) for v in np.flatnonzero(ns == 300)[:10])}):
        assert batched.models[k].status() == 0
        single = ExactTSNE(xs[k], 2.0)
        st = single.init_state(y0s[k])
        single.run(st, 2)
        for a, b in zip(batched.states[k], st):
            assert torch.equal(a, b), k
