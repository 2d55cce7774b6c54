"""The dedup of candidates whose distinct pairs are far from evenly spread, against the oracle: few
long strings (more candidates than there are pair keys), a cluster of neighbouring strings (all its
pairs in a few buckets), few queries with most of the candidates."""
import numpy as np
import pytest

import oracle
from paper_1810_08833_amd import datagen as dg
from tests.test_gpu_parity import dev, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mj():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1810_08833_amd as m
    return m


def few_long(seed, n, length):
    """Near-copies of one string: n (n - 1) / 2 pairs, each found through thousands of records."""
    rng = np.random.default_rng(seed)
    x = rng.integers(0, 4, length).astype(np.uint8)
    out = []
    for _ in range(n):
        y = x.copy()
        at = rng.integers(0, length, 9)
        y[at] = rng.integers(0, 4, 9)
        out.append(y)
    return dg.from_list(out, 4)


@pytest.mark.parametrize("n,length", [(2, 60000), (3, 60000), (9, 20000)])
def test_more_candidates_than_keys(mj, n, length):
    say("more candidates than keys", n)
    S = few_long(n, n, length)
    kw = dict(t_fixed=length // 4)
    op = oracle.make_params(6, 4, k=40, t_div=1, **kw)
    want_c, want, _ = oracle.join(S.chars, S.offsets, op)
    p = mj.Params(q=6, k=40, t_div=1, **kw)
    ctx = mj.Context()
    cand, st = mj.candidates(dev(mj, S), p, ctx=ctx)
    assert np.array_equal(cand, want_c) and st["pair_tests"] > 12288
    for mode in (0, 1, 1, 2, 2):
        ctx.set_streaming(mode)
        got, _ = mj.join(dev(mj, S), p, ctx=ctx)
        assert np.array_equal(got, want), mode


def neighbours():
    rng = np.random.default_rng(77)
    base = rng.integers(0, 4, 300).astype(np.uint8)
    strs = [rng.integers(0, 4, 300).astype(np.uint8) for _ in range(20000)]
    for i in range(5000, 5700):
        strs[i] = base.copy()
        at = rng.integers(0, 300, 4)
        strs[i][at] = rng.integers(0, 4, 4)
    return dg.from_list(strs, 4)


def test_cluster_of_neighbours(mj):
    """Most pairs are of strings 5,000 to 5,699: their dedup is left to the sort, at its speed.  (By
    buckets each of them went over its 100,000 pairs and more 64 times.)"""
    say("dedup of a cluster of neighbours")
    S = neighbours()
    want_c, want, _ = oracle.join(S.chars, S.offsets, oracle.make_params(5, 4, k=10, t_div=2))
    p = mj.Params(q=5, k=10, t_div=2)
    general = mj.Context()
    general.set_tile_emission(0)
    general.set_streaming(0)
    ctx = mj.Context()
    for _ in range(4):
        cand, st = mj.candidates(dev(mj, S), p, ctx=ctx)
        assert np.array_equal(cand, want_c)
        _, sg = mj.candidates(dev(mj, S), p, ctx=general)
    assert st["stage_ms"]["dedup"] < 4 * sg["stage_ms"]["dedup"] + 0.5
    for mode in (0, 1, 1, 1, 2, 2):
        ctx.set_streaming(mode)
        got, sj = mj.join(dev(mj, S), p, ctx=ctx)
        assert np.array_equal(got, want), mode
    assert sj["streamed"] == 2
    ctx.set_streaming(1)
    _, sj = mj.join(dev(mj, S), p, ctx=ctx)
    assert sj["streamed"] == 1 and sj["stage_ms"]["dedup"] < 4 * sg["stage_ms"]["dedup"] + 0.5


def test_few_queries_with_most_candidates(mj):
    """Four of 256 queries find 30,000 near-copies, all in one of the dedup's buckets: the next
    searches leave their dedup to the sort instead of running twice."""
    say("few queries with most of the candidates")
    rng = np.random.default_rng(78)
    base = rng.integers(0, 4, 120).astype(np.uint8)

    def copy(edits):
        x = base.copy()
        at = rng.integers(0, len(x), edits)
        x[at] = rng.integers(0, 4, edits)
        return x

    I = dg.from_list([copy(1) for _ in range(30000)] +
                     [rng.integers(0, 4, 120).astype(np.uint8) for _ in range(2000)], 4)
    Q = dg.from_list([copy(1) if i in (100, 101, 102, 103) else rng.integers(0, 4, 120).astype(np.uint8)
                      for i in range(256)], 4)
    op = oracle.make_params(5, 4, k=10, t_div=4)
    _, want = oracle.search(I.chars, I.offsets, op, Q.chars, Q.offsets, op)
    ctx = mj.Context()
    index = mj.Index(dev(mj, I), mj.Params(q=5, k=10, t_div=4), ctx=ctx)
    streamed = []
    for _ in range(5):
        got, st = index.search(dev(mj, Q), k=10)
        assert np.array_equal(got, want)
        streamed.append(st["streamed"])
    assert st["candidates"] > 80000
    assert streamed[2:] == [1, 1, 1]
    index.close()
