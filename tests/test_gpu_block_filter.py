"""Pairs that pass through the block filter before their verification (calls of 4,096 DNA pairs
or more, K >= 64) against the banded oracle: cost K - 1, K and K + 1 along the edge diagonals,
bands of less than a chunk of 448 symbols and of several, texts shorter than K blocks."""
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


@pytest.mark.parametrize("K", [64, 150, 447, 450, 1000, 2047])
def test_near_threshold(mj, K):
    say("block filter K=%d" % K)
    rng = np.random.default_rng(5000 + K)
    S, pairs = near_threshold_pairs(rng, K, 120 if K < 300 else 30 if K < 1500 else 10)
    want = oracle.verify_list(S.chars, S.offsets, oracle.make_params(4, 4, k=K), pairs)
    times = -(-4200 // len(pairs))
    got = mj.verify(dev(mj, S), mj.Params(q=4, k=K, t_div=1), np.tile(pairs, times))
    assert np.array_equal(got, np.tile(want, times))


@pytest.mark.parametrize("K", [64, 96, 150])
def test_clusters(mj, K):
    """Long copies at 1 to 8% edits, and unrelated strings: most or all pairs beyond K,
    with as many blocks missed as the filter sees in earnest."""
    say("block filter, clusters, K=%d" % K)
    S = dg.dna_long(seed=60 + K, n_clusters=12, copies=8)
    a, b = np.triu_indices(S.n, 1)
    pairs = (a.astype(np.uint64) << np.uint64(32)) | b.astype(np.uint64)
    want = oracle.verify_list(S.chars, S.offsets, oracle.make_params(5, 4, k=K), pairs)
    got = mj.verify(dev(mj, S), mj.Params(q=5, k=K, t_div=2), pairs)
    assert np.array_equal(got, want)
