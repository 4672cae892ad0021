"""Batches of more than 4,096 tiles that mix problems whose force pass runs in quarter tiles (at
most 2,048 points) with larger ones: one persistent workgroup takes tiles of both kinds in turn, on
the same LDS. Bitwise against separate runs."""
import numpy as np
import pytest
import torch

from paper_1812_09869_amd import synth
from paper_1812_09869_amd.tsne import BatchedTSNE, ExactTSNE, Schedule

pytestmark = pytest.mark.gpu


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _tiles(n):
    nb = (n + 255) // 256
    return nb * (nb + 1) // 2


def _compare(ns, chosen, iters, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    # one component: every tile holds P, so all of them are the persistent kernel's
    probs = [((rng.standard_normal((n, 3)) * 3).astype(np.float32), 8.0) for n in ns]
    y0s = [synth.embedding_init(n, seed=900 + k) for k, n in enumerate(ns)]
    assert sum(_tiles(n) for n in ns) > 4096
    print(f"\n[mixed] {len(ns)} problems, {sum(_tiles(n) for n in ns)} tiles", flush=True)
    batched = BatchedTSNE([(_t(x), p) for x, p in probs])
    batched.init_states([_t(y) for y in y0s])
    sched = Schedule(switch=2)
    batched.run(iters, sched=sched)
    assert max(m.status() for m in batched.models) == 0
    for k in chosen:
        x, p = probs[k]
        single = ExactTSNE(_t(x), p)
        st = single.init_state(_t(y0s[k]))
        single.run(st, iters, sched=sched)
        for a, b in zip(batched.states[k], st):
            assert torch.equal(a, b), (k, ns[k])


def test_small_problems_after_large_ones():
    """Large and small problems in turn: a tile of one kind follows one of the other in most of the
    512 workgroups' turns, in both orders. Every problem is compared."""
    rng = np.random.Generator(np.random.PCG64(51))
    ns = []
    for _ in range(46):
        ns += [int(rng.integers(2049, 4300)), int(rng.integers(1200, 2049))]
    _compare(ns, range(len(ns)), 4, 52)


def test_more_than_1024_problems_of_both_kinds():
    """1,030 problems, six of them large: more than the kernel keeps the table of in LDS (1,024),
    so it walks the table. The large ones, their neighbours and others on both sides of the 1,024
    boundary are compared."""
    rng = np.random.Generator(np.random.PCG64(53))
    ns = [int(v) for v in rng.integers(40, 300, 1030)]
    large = {0: 14000, 300: 2049, 700: 7000, 1023: 9000, 1025: 2300, 1029: 4097}
    for k, n in large.items():
        ns[k] = n
    chosen = sorted({min(max(k + o, 0), 1029) for k in large for o in (-1, 0, 1)} | {511})
    _compare(ns, chosen, 3, 54)
