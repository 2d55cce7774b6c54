"""Joins, candidate calls and searches on a context whose allocator has no more memory than the
general path, stage by stage, needs: whatever takes more gives way to it."""
import numpy as np
import pytest

import oracle
from paper_1810_08833_amd import datagen as dg
from tests.test_gpu_alternating import far_copies
from tests.test_gpu_bucket_sizes import near_copies
from tests.test_gpu_parity import dev, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mj():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1810_08833_amd as m
    return m


def limited(mj, limit=None):
    """An allocator that has `limit` bytes (None: all there are) and notes the most it gave out."""
    import torch
    a = mj.TorchAllocator(torch.cuda.current_device())
    give, take = a._alloc_cb, a._free_cb
    a.peak = 0
    a.refused = 0

    def alloc(nbytes, user):
        if limit is not None and sum(a.live.values()) + nbytes > limit:
            a.refused += 1
            return None
        p = give(nbytes, user)
        a.peak = max(a.peak, sum(a.live.values()))
        return p

    a.limited_cb = mj.ALLOC_FN(alloc)
    a.struct = mj.MjAllocator(a.limited_cb, take, None)
    return a


@pytest.mark.parametrize("member_filter", [-1, 1])
def test_join_within_the_general_path_memory(mj, member_filter):
    say("join, memory of the general path, member filter", member_filter)
    S = near_copies(3, 2000, 2)
    p = mj.Params(q=5, k=64, t_div=1, reps=2)
    want_c, want, _ = oracle.join(S.chars, S.offsets, oracle.make_params(5, 4, k=64, t_div=1, reps=2))

    def context(alloc):
        c = mj.Context(allocator=alloc)
        c.set_member_filter(member_filter)
        return c

    free = limited(mj)
    general = context(free)
    general.set_tile_emission(0)
    general.set_streaming(0)
    got, _ = mj.join(dev(mj, S), p, ctx=general)
    assert np.array_equal(got, want)
    general.close()
    tight = limited(mj, free.peak)
    ctx = context(tight)
    for mode in (0, 0, 1, 1, 2, 2):
        ctx.set_streaming(mode)
        got, _ = mj.join(dev(mj, S), p, ctx=ctx)
        assert np.array_equal(got, want), mode
    ctx.close()
    assert tight.refused > 0 and not tight.live
    # candidates of a fresh context
    free = limited(mj)
    general = context(free)
    general.set_tile_emission(0)
    got, _ = mj.candidates(dev(mj, S), p, ctx=general)
    assert np.array_equal(got, want_c)
    general.close()
    ctx = context(limited(mj, free.peak))
    for _ in range(2):
        got, _ = mj.candidates(dev(mj, S), p, ctx=ctx)
        assert np.array_equal(got, want_c)
    ctx.close()


def test_search_within_the_stagewise_memory(mj):
    say("search, memory of the stage-by-stage one")
    I = far_copies(32, 300, copies=6, length=1000, rate=0.01)
    Q = I.subset(np.arange(0, I.n, 2))
    op = oracle.make_params(5, 4, k=64, t_div=1)
    _, want = oracle.search(I.chars, I.offsets, op, Q.chars, Q.offsets, op)
    free = limited(mj)
    ctx = mj.Context(allocator=free)
    ctx.set_streaming(0)
    index = mj.Index(dev(mj, I), mj.Params(q=5, k=64, t_div=1), ctx=ctx)
    got, _ = index.search(dev(mj, Q), k=64)
    assert np.array_equal(got, want)
    index.close()
    ctx.close()
    ctx = mj.Context(allocator=limited(mj, free.peak))
    index = mj.Index(dev(mj, I), mj.Params(q=5, k=64, t_div=1), ctx=ctx)
    for _ in range(4):
        got, _ = index.search(dev(mj, Q), k=64)
        assert np.array_equal(got, want)
    index.close()
    ctx.close()


def test_many_queries_after_a_frequent_one(mj):
    """One query with 100 candidates a record, then 1,500 of none: the first one's rate
    does not size the second search (it took 6.8 GB)."""
    say("search, many queries after a frequent one")
    rng = np.random.default_rng(35)
    base = rng.integers(0, 4, 120).astype(np.uint8)
    I = dg.from_list([base] * 6000 + [rng.integers(0, 4, 120).astype(np.uint8) for _ in range(500)], 4)
    rest = dg.from_list([rng.integers(0, 4, 120).astype(np.uint8) for _ in range(1500)], 4)
    op = oracle.make_params(5, 4, k=10, t_div=1)
    alloc = limited(mj)
    ctx = mj.Context(allocator=alloc)
    index = mj.Index(dev(mj, I), mj.Params(q=5, k=10, t_div=1), ctx=ctx)
    one = dg.from_list([base], 4)
    for _ in range(2):
        got, st = index.search(dev(mj, one), k=10)
        assert np.array_equal(got, np.arange(6000, dtype=np.uint64)) and st["candidates"] >= 6000
    assert st["streamed"] == 1
    _, want = oracle.search(I.chars, I.offsets, op, rest.chars, rest.offsets, op)
    for _ in range(2):
        got, _ = index.search(dev(mj, rest), k=10)
        assert np.array_equal(got, want)
    assert alloc.peak < 1 << 30
    index.close()
    ctx.close()


@pytest.mark.parametrize("n,table", [(0, False), (1, False), (37, True), (1000, False)])
def test_index_bytes(mj, n, table):
    """mj_index_bytes is what freeing the index gives back to the allocator."""
    import torch
    say("index bytes", n, table)
    rng = np.random.default_rng(n)
    I = dg.from_list([rng.integers(0, 4, int(rng.integers(100, 500))).astype(np.uint8) for _ in range(n)], 4)
    alloc = limited(mj)
    ctx = mj.Context(allocator=alloc)
    pi = torch.from_numpy(rng.permutation(4 ** 5).astype(np.int64)).cuda() if table else None
    index = mj.Index(dev(mj, I), mj.Params(q=5, k=10, t_div=1, pi_table=pi), ctx=ctx)
    with_index, said = sum(alloc.live.values()), index.device_bytes
    index.close()
    assert with_index - sum(alloc.live.values()) == said > 0
    ctx.close()
