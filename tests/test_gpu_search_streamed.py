"""Repeated searches of one context (stage by stage, then sized by the last one's rates) over an
index with its key directory, against the oracle: few and many records, frequent keys, queries
that need more room than the last ones did, and queries without candidates; and joins at both
sides of the sizes up to which small calls take single launches."""
import numpy as np
import pytest

import oracle
from paper_1810_08833_amd import datagen as dg
from tests.test_gpu_buckets import shared_segments, tandem
from tests.test_gpu_parity import dev, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mj():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1810_08833_amd as m
    return m


def altered(S, ids, seed):
    """Strings `ids` of S, each with a few substitutions."""
    rng = np.random.default_rng(seed)
    out = []
    for i in ids:
        x = S.get(i).copy()
        at = rng.integers(0, len(x), 5)
        x[at] = (x[at] + rng.integers(1, 4, 5)) % 4
        out.append(x)
    return dg.from_list(out, 4)


INDEXES = {
    "one_string": lambda: shared_segments(21, 1, 1),
    "shared": lambda: shared_segments(22, 60, 5),
    "frequent_keys": lambda: tandem(23, 200),
    "many": lambda: shared_segments(24, 2500, 2),
}


@pytest.mark.parametrize("name", sorted(INDEXES))
def test_repeated_searches(mj, name):
    import torch
    say("repeated searches", name)
    I = INDEXES[name]()
    ctx = mj.Context()
    index = mj.Index(dev(mj, I), mj.Params(q=5, k=30, t_div=2), ctx=ctx)
    op = oracle.make_params(5, 4, k=30, t_div=2)
    few = altered(I, [0], 31)
    more = altered(I, np.arange(min(I.n, 40)), 32)
    all_ = altered(I, np.arange(I.n), 33)
    none = dg.from_list([np.zeros(7, np.uint8)], 4)
    for step, Q in enumerate((few, few, more, all_, all_, none, few, all_)):
        _, want = oracle.search(I.chars, I.offsets, op, Q.chars, Q.offsets, op)
        kq = torch.full((Q.n,), 30, dtype=torch.int32, device="cuda")
        got, st = index.search(dev(mj, Q), k_per_query=kq)
        assert np.array_equal(got, want), step
        if step == 1:
            assert st["streamed"] == 1
    index.close()


# tile scans of one launch take up to 8 chunks of all repetitions
@pytest.mark.parametrize("reps", [1, 8, 9])
def test_small_join_repetitions(mj, reps):
    say("small joins, repetitions", reps)
    S = shared_segments(40 + reps, 20, 4)
    want_c, want, _ = oracle.join(S.chars, S.offsets, oracle.make_params(5, 4, k=30, t_div=2, reps=reps))
    ctx = mj.Context()
    for _ in range(3):
        got, _ = mj.join(dev(mj, S), mj.Params(q=5, k=30, t_div=2, reps=reps), ctx=ctx)
        assert np.array_equal(got, want)


# one launch orders up to 8192 candidates and one compacts up to 32768
@pytest.mark.parametrize("n", [127, 129, 130, 256, 258])
def test_candidates_around_small_calls(mj, n):
    say("small calls, strings", n)
    S = tandem(50 + n, n)
    want_c, want, _ = oracle.join(S.chars, S.offsets, oracle.make_params(5, 4, k=30, t_div=2))
    ctx = mj.Context()
    for _ in range(3):
        got, st = mj.join(dev(mj, S), mj.Params(q=5, k=30, t_div=2), ctx=ctx)
        assert st["candidates"] == len(want_c) and np.array_equal(got, want)
