"""Limits of a search hold for a repeated one too, which sizes its stages by the last one's rates."""
import numpy as np
import pytest

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


def test_pair_tests_beyond_2_31(mj):
    """Strings 0010010..0 of 20 symbols and queries of 21: with 1 the least symbol's hash, every
    query shares the partitions 00 and 100 with every string, and no pair passes K = 0."""
    import torch
    say("2.2e9 pair tests")
    pi = torch.tensor([5, 1, 8, 9], dtype=torch.int64, device="cuda")

    def strings(n, m):
        x = np.zeros((n, m), np.uint8)
        x[:, 2] = x[:, 5] = 1
        return dg.from_list(list(x), 4)

    n = 33000
    index = mj.Index(dev(mj, strings(n, 20)), mj.Params(q=1, k=0, t_fixed=8, pi_table=pi), ctx=mj.Context())
    got, st = index.search(dev(mj, strings(1, 21)), k=0)
    assert len(got) == 0 and st["pair_tests"] == 2 * n
    got, st = index.search(dev(mj, strings(1000, 21)), k=0)
    assert len(got) == 0 and st["pair_tests"] == 2 * n * 1000 and st["streamed"] == 1
    for _ in range(2):
        with pytest.raises(mj.MinJoinError) as e:
            index.search(dev(mj, strings(n, 21)), k=0)
        assert e.value.status == mj.MJ_ECAPACITY and "2^31" in str(e.value)
    got, st = index.search(dev(mj, strings(1000, 21)), k=0)
    assert len(got) == 0 and st["pair_tests"] == 2 * n * 1000
    index.close()
