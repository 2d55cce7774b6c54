"""The skewed band (the batched verifier's layout for small calls) against the banded oracle,
at the edges of its classes: bands of up to 32 W (G - 2) diagonals for G lanes a half and W
words a lane, texts of one column up, and both symbol widths of a plane word's neighbours."""
import numpy as np
import pytest

import oracle
from paper_1810_08833_amd import datagen as dg
from tests.test_gpu_parity import dev, near_threshold_pairs, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mj():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1810_08833_amd as m
    return m


# the largest K of each class (G, W) and the one after it, and the largest K there is
@pytest.mark.parametrize("K", [2, 63, 64, 65, 95, 97, 192, 193, 448, 449, 896, 897, 1344, 1345, 2047])
def test_class_edges(mj, K):
    say("skewed band K=%d" % K)
    rng = np.random.default_rng(3000 + K)
    S, pairs = near_threshold_pairs(rng, K, 120 if K < 300 else 30 if K < 1000 else 10)
    got = mj.verify(dev(mj, S), mj.Params(q=4, k=K, t_div=1), pairs)
    want = oracle.verify_list(S.chars, S.offsets, oracle.make_params(4, 4, k=K), pairs)
    assert np.array_equal(got, want)
    assert 0 < want.sum() < len(want)


@pytest.mark.parametrize("sigma", [2, 4, 25, 37, 200])
def test_ragged_lengths_and_alphabets(mj, sigma):
    """Texts of 1 to 200 symbols (halves of no columns, bands wider than the strings, the
    first and the last string of the collection) and all four plane counts."""
    say("skewed band, short texts, sigma=%d" % sigma)
    rng = np.random.default_rng(4000 + sigma)
    strs = []
    for m in list(range(1, 70)) + [95, 96, 97, 127, 128, 129, 190, 200]:
        x = rng.integers(0, sigma, m).astype(np.uint8)
        strs += [x, dg.mutate(rng, x, rng.uniform(0, 0.5), sigma)]
    S = dg.from_list(strs, sigma)
    pairs = np.array([(2 * i << 32) | (2 * j + 1) for i in range(len(strs) // 2)
                      for j in {i, max(0, i - 1), min(len(strs) // 2 - 1, i + 3)}], dtype=np.uint64)
    for K in (0, 1, 5, 31, 64, 130):
        got = mj.verify(dev(mj, S), mj.Params(q=2, k=K, t_div=1), pairs)
        want = oracle.verify_list(S.chars, S.offsets, oracle.make_params(2, sigma, k=K), pairs)
        assert np.array_equal(got, want), K
