"""Grouping, pair tests and dedup by LDS buckets against the oracle and against the general path
(taken by a context that tests every join's large groups by tile pairs): slots of more records
than a slot of the bucket holds, buckets of more distinct pairs than the dedup's table, one
bucket and many, repeated calls (stage by stage, streamed, captured)."""
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


def shared_segments(seed, groups, copies, seg=150, parts=4):
    """Random strings of `parts` segments, group g's strings with the same segment g mod parts."""
    rng = np.random.default_rng(seed)
    strs = []
    for g in range(groups):
        common = rng.integers(0, 4, seg).astype(np.uint8)
        for _ in range(copies):
            x = rng.integers(0, 4, seg * parts).astype(np.uint8)
            at = (g % parts) * seg
            x[at:at + seg] = common
            strs.append(x)
    order = rng.permutation(len(strs))
    return dg.from_list([strs[i] for i in order], 4)


def tandem(seed, n, unit=40, times=12):
    """Repeats of one unit at random phases: a string has many records of one key, a pair of
    strings many candidates."""
    rng = np.random.default_rng(seed)
    u = rng.integers(0, 4, unit).astype(np.uint8)
    strs = []
    for _ in range(n):
        x = np.tile(u, times + 2)[int(rng.integers(0, unit)):][:unit * times].copy()
        x[rng.integers(0, len(x), 6)] = rng.integers(0, 4, 6)
        strs.append(x)
    return dg.from_list(strs, 4)


INPUTS = {
    "three_strings": lambda: shared_segments(1, 1, 3),
    "groups_of_31_to_33": lambda: dg.from_list(sum(([s.get(i) for i in range(s.n)] for s in (
        shared_segments(2, 1, 31), shared_segments(3, 1, 32), shared_segments(4, 1, 33))), []), 4),
    "hundred_a_group": lambda: shared_segments(5, 4, 100),
    "tandem": lambda: tandem(6, 60),
    "groups_of_62_to_65": lambda: dg.from_list(sum(([s.get(i) for i in range(s.n)] for s in (
        shared_segments(8, 1, 62), shared_segments(9, 1, 63), shared_segments(10, 1, 64),
        shared_segments(11, 1, 65))), []), 4),
    "many_buckets": lambda: shared_segments(7, 300, 10),
}


@pytest.mark.parametrize("name", sorted(INPUTS))
def test_buckets_match_oracle(mj, name):
    say("buckets", name)
    S = INPUTS[name]()
    want_c, want, _ = oracle.join(S.chars, S.offsets, oracle.make_params(5, 4, k=30, t_div=2))
    p = mj.Params(q=5, k=30, t_div=2)
    general = mj.Context()
    general.set_tile_emission(0)
    ctx = mj.Context()
    cand, st = mj.candidates(dev(mj, S), p, ctx=ctx)
    cand_g, st_g = mj.candidates(dev(mj, S), p, ctx=general)
    assert np.array_equal(cand, want_c) and np.array_equal(cand_g, want_c)
    for f in ("records", "groups", "pair_tests", "candidates"):
        assert st[f] == st_g[f], f
    for mode in (0, 1, 1, 2, 2):
        ctx.set_streaming(mode)
        got, sj = mj.join(dev(mj, S), p, ctx=ctx)
        assert np.array_equal(got, want), mode
        for f in ("records", "groups", "pair_tests", "candidates"):
            assert sj[f] == st_g[f], (mode, f)
    # another collection of the same parameters: capacities and choices of the last one
    T = INPUTS["hundred_a_group"]()
    got, _ = mj.join(dev(mj, T), p, ctx=ctx)
    _, want, _ = oracle.join(T.chars, T.offsets, oracle.make_params(5, 4, k=30, t_div=2))
    assert np.array_equal(got, want)


@pytest.mark.parametrize("name", sorted(INPUTS))
def test_member_buckets_match_oracle(mj, name):
    """The same over the records that the member filter keeps (nearly all of them members), with
    one distinct bucket limit that keeps every record."""
    say("member_buckets", name)
    S = INPUTS[name]()
    want_c, want, _ = oracle.join(S.chars, S.offsets, oracle.make_params(5, 4, k=30, t_div=2))
    p = mj.Params(q=5, k=30, t_div=2)
    for limit in (0, 1):
        ctx = mj.Context()
        ctx.set_member_filter(1, limit)
        cand, st = mj.candidates(dev(mj, S), p, ctx=ctx)
        assert st["member_filter"] == 1 and np.array_equal(cand, want_c)
        for mode in (0, 1, 1, 2, 2):
            ctx.set_streaming(mode)
            got, sj = mj.join(dev(mj, S), p, ctx=ctx)
            assert np.array_equal(got, want), mode
            for f in ("records", "groups", "pair_tests", "candidates"):
                assert sj[f] == st[f], (mode, f)
    plain, sp = mj.candidates(dev(mj, S), p)
    assert np.array_equal(plain, want_c)
    for f in ("records", "groups", "pair_tests", "candidates"):
        assert sp[f] == st[f], f


def test_more_candidates_than_records(mj):
    """A first join with more candidates than the room its tests start with (65,536, or one a
    record): strings of one repeated unit."""
    say("candidates beyond the first room")
    S = tandem(12, 420)
    want_c, want, _ = oracle.join(S.chars, S.offsets, oracle.make_params(5, 4, k=30, t_div=2))
    p = mj.Params(q=5, k=30, t_div=2)
    general = mj.Context()
    general.set_tile_emission(0)
    _, st_g = mj.candidates(dev(mj, S), p, ctx=general)
    ctx = mj.Context()
    cand, st = mj.candidates(dev(mj, S), p, ctx=ctx)
    assert np.array_equal(cand, want_c) and st["pair_tests"] == st_g["pair_tests"] > 65536
    for limit in (1024, 1 << 20):  # tile pairs beyond a pass: the general path, in passes
        ctx = mj.Context()
        ctx.set_pair_test_pass(limit)
        for _ in range(2):
            got, _ = mj.join(dev(mj, S), p, ctx=ctx)
            assert np.array_equal(got, want)
