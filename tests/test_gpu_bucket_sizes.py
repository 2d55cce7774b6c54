"""Joins whose records nearly all share their keys, at the sizes where a bucket of the usual record
count holds more members than its LDS: smaller buckets, found once and kept for the next calls."""
import numpy as np
import pytest

import oracle
from paper_1810_08833_amd import datagen as dg
from tests.test_gpu_buckets import shared_segments
from tests.test_gpu_parity import dev, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mj():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1810_08833_amd as m
    return m


def near_copies(seed, clusters, copies, length=2000, edits=3):
    rng = np.random.default_rng(seed)
    strs = []
    for _ in range(clusters):
        x = rng.integers(0, 4, length).astype(np.uint8)
        for _ in range(copies):
            y = x.copy()
            at = rng.integers(0, length, edits)
            y[at] = rng.integers(0, 4, edits)
            strs.append(y)
    return dg.from_list(strs, 4)


# records: just below one bucket's, four buckets' and 512 buckets' size (where the smaller ones
# need a second radix pass, and where they do not)
@pytest.mark.parametrize("clusters,buckets", [(20, 1), (80, 4), (10500, 512)])
def test_mostly_members(mj, clusters, buckets):
    say("mostly members, clusters", clusters)
    S = near_copies(90 + clusters, clusters, 3, 2000, 2)
    want_c, want, _ = oracle.join(S.chars, S.offsets, oracle.make_params(5, 4, k=30, t_div=2))
    p = mj.Params(q=5, k=30, t_div=2)
    ctx = mj.Context()
    for call in range(3):
        cand, st = mj.candidates(dev(mj, S), p, ctx=ctx)
        assert np.array_equal(cand, want_c)
        assert 900 * buckets < st["records"] <= 1024 * buckets
        # the pair tests that did not fit run a second time, once
        assert st["kernel_launches"]["emit"] == (2 if call == 0 else 1)
    general = mj.Context()
    general.set_tile_emission(0)
    _, sg = mj.candidates(dev(mj, S), p, ctx=general)
    for mode in (0, 1, 1, 2, 2):
        ctx.set_streaming(mode)
        got, sj = mj.join(dev(mj, S), p, ctx=ctx)
        assert np.array_equal(got, want), mode
        for f in ("records", "groups", "pair_tests", "candidates"):
            assert sj[f] == sg[f], (mode, f)
    assert sj["streamed"] == 2
    # few of the records members again, then a fresh context's first calls by joins
    T = dg.from_list([np.random.default_rng(i).integers(0, 4, 2000).astype(np.uint8) for i in range(60)]
                     + [S.get(0), S.get(1)], 4)
    _, want_t, _ = oracle.join(T.chars, T.offsets, oracle.make_params(5, 4, k=30, t_div=2))
    other = mj.Context()
    for c, A, w in ((ctx, T, want_t), (ctx, S, want), (other, T, want_t), (other, S, want), (other, S, want)):
        c.set_streaming(1)
        got, _ = mj.join(dev(mj, A), p, ctx=c)
        assert np.array_equal(got, w)


# tile pairs of which all record pairs are candidates: one, whole and partly filled tiles, several
@pytest.mark.parametrize("copies", [64, 65, 68, 69, 127, 128, 129, 193])
def test_full_tile_pairs(mj, copies):
    say("full tile pairs", copies)
    S = shared_segments(200 + copies, 1, copies)
    want_c, want, _ = oracle.join(S.chars, S.offsets, oracle.make_params(5, 4, k=30, t_div=2))
    p = mj.Params(q=5, k=30, t_div=2)
    assert len(want_c) >= copies * (copies - 1) // 2
    ctx = mj.Context()
    got, _ = mj.candidates(dev(mj, S), p, ctx=ctx)
    assert np.array_equal(got, want_c) and ctx.grouping()[0]
    for _ in range(2):
        got, _ = mj.join(dev(mj, S), p, ctx=ctx)
        assert np.array_equal(got, want)
