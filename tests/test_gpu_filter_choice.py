"""The block filter is timed with the verifier's other choices: it stays off where most pairs are
within K, and comes back for other pairs; the results are the oracle's either way."""
import numpy as np
import pytest

import oracle
from paper_1810_08833_amd import datagen as dg
from tests.test_gpu_alternating import far_copies
from tests.test_gpu_parity import dev, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mj():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1810_08833_amd as m
    return m


def copies(n, per, length, rate, seed=1):
    """n strings on the GPU, clusters of `per` copies with substitutions only."""
    import torch
    import paper_1810_08833_amd as mj
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    x = torch.randint(0, 4, (-(-n // per), length), generator=g, device="cuda", dtype=torch.uint8)
    x = x.repeat_interleave(per, 0)[:n].reshape(-1)
    edit = torch.rand(x.numel(), generator=g, device="cuda") < rate
    other = torch.randint(0, 4, (x.numel(),), generator=g, device="cuda", dtype=torch.uint8)
    return mj.DeviceStrings(torch.where(edit, other, x), torch.arange(n + 1, device="cuda") * length, 4)


def test_all_pairs_within_k(mj):
    """Every pair is within K: the filter and the best bands after it took 1.1 times the time of the
    best of three fixed choices without it."""
    say("filter choice: all within K")
    S = copies(48000, 8, 1250, 0.03)
    best, want = 1e9, None
    for lanes in (1, 2, -2):
        ctx = mj.Context()
        p = mj.Params(q=5, k=100, t_div=2, verify_lanes=lanes)
        for _ in range(7):
            want, st = mj.join(S, p, ctx=ctx)
            best = min(best, st["stage_ms"]["verify"])
    ctx = mj.Context()
    times = []
    for _ in range(9):
        got, st = mj.join(S, mj.Params(q=5, k=100, t_div=2), ctx=ctx)
        times.append(st["stage_ms"]["verify"])
    assert np.array_equal(got, want) and len(got) > 0.9 * st["candidates"] > 100000
    print("lanes %.3f ms, chosen" % best, ["%.3f" % t for t in times], flush=True)
    assert min(times[2:]) < 1.05 * best


def test_other_pairs_after_those_within_k(mj):
    """Near pairs first, then far ones, longer strings, searches and pair lists on one context."""
    say("filter choice: near, then far")
    p = mj.Params(q=5, k=64, t_div=2)
    op = oracle.make_params(5, 4, k=64, t_div=2)
    ctx = mj.Context()
    near = far_copies(51, 250, copies=8, length=900, rate=0.005)
    far = far_copies(52, 420, copies=12, length=1000, rate=0.03)
    long_far = far_copies(53, 700, copies=12, length=2200, rate=0.05)
    for S in (near, near, far, far, near, long_far, long_far, near):
        want_c, want, _ = oracle.join(S.chars, S.offsets, op)
        got, st = mj.join(dev(mj, S), p, ctx=ctx)
        assert np.array_equal(got, want) and st["candidates"] == len(want_c) > 4096
        flags = mj.verify(dev(mj, S), p, want_c, ctx=ctx)
        assert np.array_equal(want_c[flags], want)
    # far pairs of long strings walk hardly a column
    got, st = mj.join(dev(mj, long_far), p, ctx=ctx)
    assert st["band_cells"] < 65 * st["candidates"]
    index = mj.Index(dev(mj, near), p, ctx=ctx)
    for Q in (near, near.subset(np.arange(0, near.n, 2)), far, near):
        _, want = oracle.search(near.chars, near.offsets, op, Q.chars, Q.offsets, op)
        got, _ = index.search(dev(mj, Q), k=64)
        assert np.array_equal(got, want)
    index.close()
