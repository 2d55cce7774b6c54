"""The way each call takes: results alone do not show it, since whatever does not fit the LDS
buckets, a streamed call's room or the block filter gives way to a path with the same results."""
import numpy as np
import pytest

import oracle
from paper_1810_08833_amd import datagen as dg
from tests.test_gpu_alternating import far_copies
from tests.test_gpu_bucket_sizes import near_copies
from tests.test_gpu_buckets import INPUTS, tandem
from tests.test_gpu_dedup import few_long, neighbours
from tests.test_gpu_memory import limited
from tests.test_gpu_parity import dev, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mj():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1810_08833_amd as m
    return m


@pytest.mark.parametrize("members", [False, True])
@pytest.mark.parametrize("name", sorted(INPUTS))
def test_buckets_taken(mj, name, members):
    say("buckets taken", name, members)
    S = INPUTS[name]()
    p = mj.Params(q=5, k=30, t_div=2)
    ctx = mj.Context()
    if members:
        ctx.set_member_filter(1)
    _, st = mj.candidates(dev(mj, S), p, ctx=ctx)
    assert ctx.grouping() == (True, True, 0)
    for mode, streamed in ((0, 0), (1, 1), (1, 1), (2, 2), (2, 2)):
        ctx.set_streaming(mode)
        _, sj = mj.join(dev(mj, S), p, ctx=ctx)
        assert sj["streamed"] == streamed and ctx.grouping() == (True, True, 0), mode
        assert sj["member_filter"] == (1 if members else 0)
    ctx.set_tile_emission(0)
    ctx.set_streaming(0)
    mj.join(dev(mj, S), p, ctx=ctx)
    assert ctx.grouping() == (False, False, 0)


def test_more_tests_than_a_pass(mj):
    say("left: tests")
    S = tandem(12, 420)
    ctx = mj.Context()
    ctx.set_pair_test_pass(1024)
    p = mj.Params(q=5, k=30, t_div=2)
    mj.candidates(dev(mj, S), p, ctx=ctx)
    assert ctx.grouping() == (False, False, mj.LEFT_TESTS)
    mj.candidates(dev(mj, S), p, ctx=ctx)  # not tried again at once
    assert ctx.grouping() == (False, False, 0)


def test_parameters_in_turn(mj):
    """Calls of several parameters on one context: what each found holds for its next call."""
    say("parameters in turn")
    S = tandem(12, 420)
    ctx = mj.Context()
    ctx.set_pair_test_pass(1024)
    for call in range(3):
        for k in (28, 29, 30, 31, 32):
            mj.candidates(dev(mj, S), mj.Params(q=5, k=k, t_div=2), ctx=ctx)
            assert ctx.grouping() == (False, False, 0 if call else mj.LEFT_TESTS)


def test_candidates_beyond_the_records(mj):
    """More candidates than the first call has room for: its tests run twice, the next calls' once,
    and calls with few candidates follow."""
    say("candidates beyond the records")
    S, few = tandem(12, 420), near_copies(72, 3, 2)
    p = mj.Params(q=5, k=30, t_div=2)
    ctx = mj.Context()
    for emits in (2, 1, 1):
        _, st = mj.candidates(dev(mj, S), p, ctx=ctx)
        assert st["kernel_launches"]["emit"] == emits and ctx.grouping()[0]
    _, want, _ = oracle.join(few.chars, few.offsets, oracle.make_params(5, 4, k=30, t_div=2))
    got, _ = mj.join(dev(mj, few), p, ctx=ctx)
    assert np.array_equal(got, want)


def test_pairs_of_one_dedup_bucket(mj):
    say("left: dedup")
    S = neighbours()
    p = mj.Params(q=5, k=10, t_div=2)
    ctx = mj.Context()
    mj.candidates(dev(mj, S), p, ctx=ctx)
    assert ctx.grouping() == (True, False, mj.LEFT_DEDUP)
    for streamed in (0, 1, 1):
        _, st = mj.join(dev(mj, S), p, ctx=ctx)
        assert st["streamed"] == streamed and ctx.grouping() == (True, False, 0)


def test_more_candidates_than_keys(mj):
    say("dedup of few strings by the sort")
    ctx = mj.Context()
    mj.candidates(dev(mj, few_long(2, 2, 60000)), mj.Params(q=6, k=40, t_fixed=15000), ctx=ctx)
    assert ctx.grouping() == (True, False, 0)


def test_more_members_than_expected(mj):
    """Homopolymers have one record a string, so a join of other strings after them has far more
    records than the streamed one's buckets are made for: stage by stage, in buckets all the same."""
    say("left: members")
    homo = dg.from_list([np.full(2000, i % 4, np.uint8) for i in range(40)], 4)
    S = near_copies(70, 20, 9)
    p = mj.Params(q=5, k=30, t_div=2)
    _, want, _ = oracle.join(S.chars, S.offsets, oracle.make_params(5, 4, k=30, t_div=2))
    ctx = mj.Context()
    for _ in range(2):
        mj.join(dev(mj, homo), p, ctx=ctx)
    got, st = mj.join(dev(mj, S), p, ctx=ctx)
    assert np.array_equal(got, want) and 768 < st["records"] < 4096
    assert st["streamed"] == 0 and ctx.grouping() == (True, True, mj.LEFT_MEMBERS)
    got, st = mj.join(dev(mj, S), p, ctx=ctx)
    assert np.array_equal(got, want)
    assert st["streamed"] == 1 and ctx.grouping() == (True, True, 0)


def test_no_memory_for_buckets(mj):
    say("left: memory")
    S = near_copies(3, 2000, 2)
    p = mj.Params(q=5, k=64, t_div=1, reps=2)
    free = limited(mj)
    general = mj.Context(allocator=free)
    general.set_tile_emission(0)
    general.set_streaming(0)
    mj.join(dev(mj, S), p, ctx=general)
    general.close()
    ctx = mj.Context(allocator=limited(mj, free.peak))
    mj.join(dev(mj, S), p, ctx=ctx)
    assert ctx.grouping() == (False, False, mj.LEFT_MEMORY)
    ctx.close()


def test_buckets_after_a_join_too_large_for_them(mj):
    """More than 2^23 records without the member filter are sorted; the next, smaller join of the
    same parameters is in buckets at once."""
    say("small join after one too large for buckets")
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    n, m = 120000, 1000
    chars = torch.randint(0, 4, (n * m,), generator=gen, device="cuda", dtype=torch.uint8)
    big = mj.DeviceStrings(chars, torch.arange(n + 1, device="cuda") * m, 4)
    S = near_copies(71, 40, 6, 1000)
    p = mj.Params(q=10, k=10, t_fixed=70)
    ctx = mj.Context()
    ctx.set_member_filter(-1)
    _, st = mj.join(big, p, ctx=ctx)
    assert st["records"] > 1 << 23 and ctx.grouping() == (False, False, 0)
    _, want, _ = oracle.join(S.chars, S.offsets, oracle.make_params(10, 4, k=10, t_fixed=70))
    got, _ = mj.join(dev(mj, S), p, ctx=ctx)
    assert np.array_equal(got, want) and ctx.grouping()[0]


def test_block_filter_rejects(mj):
    """Candidates all far apart: the filter leaves none, so no band walks a column, stage by stage
    and streamed."""
    say("block filter rejects")
    S = far_copies(9, 600, rate=0.05)
    ctx = mj.Context()
    for _ in range(3):
        _, st = mj.join(dev(mj, S), mj.Params(q=5, k=64, t_div=2), ctx=ctx)
        assert st["candidates"] >= 4096
        assert st["band_cells"] < 65 * st["candidates"]  # less than a column each
    _, plain = mj.join(dev(mj, S), mj.Params(q=5, k=64, t_div=2, verify_lanes=8), ctx=ctx)
    assert plain["band_cells"] > 100 * 65 * plain["candidates"]
