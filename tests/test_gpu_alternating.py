"""Small and large calls of the same parameters on one context: what the last call found must not
size the next one by its own count."""
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


def far_copies(seed, clusters, copies=12, length=2000, sigma=4, rate=0.04):
    """Copies of hidden strings, each with `rate` edits of its own: pairs of a cluster share
    partitions but most are more than twice `rate` apart."""
    rng = np.random.default_rng(seed)
    strs = []
    for _ in range(clusters):
        x = rng.integers(0, sigma, length).astype(np.uint8)
        strs += [dg.mutate(rng, x, rate, sigma) for _ in range(copies)]
    return dg.from_list(strs, sigma)


def test_small_and_large_joins(mj):
    """The block filter and the launches for many pairs serve the large joins between small ones:
    the filter shows in the columns the bands walk."""
    say("small and large joins in turn")
    p = mj.Params(q=5, k=64, t_div=2)
    op = oracle.make_params(5, 4, k=64, t_div=2)
    near = far_copies(3, 20, rate=0.01)
    small = far_copies(1, 1, rate=0.02)
    far = far_copies(2, 430)
    large = dg.from_list([S.get(i) for S in (near, far) for i in range(S.n)], 4)
    want_s, want_l = (oracle.join(S.chars, S.offsets, op)[1] for S in (small, large))
    _, unfiltered = mj.join(dev(mj, large), mj.Params(q=5, k=64, t_div=2, verify_lanes=8), ctx=mj.Context())
    assert unfiltered["candidates"] > 8192
    ctx = mj.Context()
    for call in range(3):
        got, _ = mj.join(dev(mj, small), p, ctx=ctx)
        assert np.array_equal(got, want_s)
        got, st = mj.join(dev(mj, large), p, ctx=ctx)
        assert np.array_equal(got, want_l)
        assert st["candidates"] == unfiltered["candidates"]
        if call:  # (the first large one may go stage by stage)
            assert st["streamed"] == 1
        assert 2 * st["band_cells"] < unfiltered["band_cells"], call


@pytest.mark.parametrize("sigma,rate,tunes", [(25, 0.01, True), (4, 0.01, True), (4, 0.08, False)])
def test_large_searches_after_a_small_one(mj, sigma, rate, tunes):
    """The verifier's choices are timed once a search has pairs enough, also where the context's
    first searches had few, and where the block filter leaves few the searches stay streamed."""
    say("large searches after a small one", sigma, rate)
    I = far_copies(5 + sigma, 900, copies=6, length=700, sigma=sigma, rate=rate)
    kw = dict(t_div=2)
    ctx = mj.Context()
    index = mj.Index(dev(mj, I), mj.Params(q=4, k=64, **kw), ctx=ctx)
    op = oracle.make_params(4, sigma, k=64, **kw)
    few = I.subset([0])
    many = I.subset(np.arange(0, I.n, 3))
    streamed = []
    for Q in (few, few, many, many, many, few, many):
        _, want = oracle.search(I.chars, I.offsets, op, Q.chars, Q.offsets, op)
        got, st = index.search(dev(mj, Q), k=64)
        assert np.array_equal(got, want)
        streamed.append(st["streamed"])
    assert st["candidates"] > 4096
    assert streamed[:2] == [0, 1]
    if tunes:
        assert streamed[2] == 0
    assert streamed[4:] == [1, 1, 1]
    index.close()
