"""Batches of more than 6,000 tiles that mix problems whose force pass runs in quarter tiles (at
most 2,048 points) with larger ones, whose tiles are the most: one persistent workgroup takes tiles
of both kinds in turn, on the same LDS. Bitwise against separate runs. And batches at the lines
between the launches."""
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
    assert sum(_tiles(n) for n in ns) > 6000
    assert 2 * sum(_tiles(n) for n in ns if n <= 2048) < sum(_tiles(n) for n in ns)
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
    for _ in range(62):
        ns += [int(rng.integers(2049, 4300)), int(rng.integers(1200, 2049))]
    _compare(ns, range(len(ns)), 4, 52)


def test_more_than_1024_problems_of_both_kinds():
    """1,030 problems, six of them large: more than the kernel keeps the table of in LDS (1,024),
    so it walks the table. The large ones, their neighbours and others on both sides of the 1,024
    boundary are compared."""
    rng = np.random.Generator(np.random.PCG64(53))
    ns = [int(v) for v in rng.integers(40, 300, 1030)]
    large = {0: 20000, 300: 2049, 700: 8000, 1023: 9000, 1025: 6000, 1029: 4097}
    for k, n in large.items():
        ns[k] = n
    chosen = sorted({min(max(k + o, 0), 1029) for k in large for o in (-1, 0, 1)} | {511})
    _compare(ns, chosen, 3, 54)


@pytest.mark.parametrize("ns", [
    [2000] * 7,                  # 1,008 units, one to a workgroup
    [2000] * 8,                  # 1,152, two to a workgroup
    [2000] * 11 + [700],         # 1,608: whole tiles' launch
    [2040] * 150 + [20000],      # 8,560 tiles, 5,400 of them small problems': one launch
], ids=["one", "two", "four", "most"])
def test_lines_between_launches(ns):
    rng = np.random.Generator(np.random.PCG64(len(ns)))
    probs = [((rng.standard_normal((n, 3)) * 3).astype(np.float32), 8.0) for n in ns]
    y0s = [synth.embedding_init(n, seed=70 + k) for k, n in enumerate(ns)]
    print(f"\n[mixed] {len(ns)} problems, {sum(_tiles(n) for n in ns)} tiles", flush=True)
    batched = BatchedTSNE([(_t(x), p) for x, p in probs])
    batched.init_states([_t(y) for y in y0s])
    batched.run(2, sched=Schedule(switch=1))
    assert max(m.status() for m in batched.models) == 0
    for k in sorted({0, 1, len(ns) // 2, len(ns) - 2, len(ns) - 1}):
        x, p = probs[k]
        single = ExactTSNE(_t(x), p)
        st = single.init_state(_t(y0s[k]))
        single.run(st, 2, sched=Schedule(switch=1))
        for a, b in zip(batched.states[k], st):
            assert torch.equal(a, b), (k, ns[k])


@pytest.mark.parametrize("n", [19201, 20001])
def test_two_streams_against_one_launch(n):
    """A problem of more than 2,850 tiles runs its two kinds of tile on two streams, a batch of it
    alone in one launch: bitwise the same, with a ragged last row block and zero tiles."""
    rng = np.random.Generator(np.random.PCG64(n))
    x = rng.standard_normal((n, 4)) + 40.0 * rng.standard_normal((12, 4))[rng.integers(0, 12, n)]
    x = _t(x.astype(np.float32))
    y0 = _t(synth.embedding_init(n, seed=n))
    print(f"\n[mixed] n={n}, {_tiles(n)} tiles", flush=True)
    single = ExactTSNE(x, 12.0)
    st = single.init_state(y0)
    single.run(st, 3, sched=Schedule(switch=2))
    batched = BatchedTSNE([(x, 12.0)])
    batched.init_states([y0])
    batched.run(3, sched=Schedule(switch=2))
    assert single.status() == 0 and batched.models[0].status() == 0
    for a, b in zip(batched.states[0], st):
        assert torch.equal(a, b)
