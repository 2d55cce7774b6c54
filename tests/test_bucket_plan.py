"""The dedup's choice of LDS buckets (csrc/bucket_plan.h), walked on the CPU: the bits that number
a bucket and those its table holds are shift counts in the kernels, so both have to stay in range
for every number of strings and candidates, few strings with many candidates among them."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1810_08833_amd", "csrc")
MAIN = r"""
#include "bucket_plan.h"
#include <stdio.h>
int main() {
    long long e, u; int a, b;
    while (scanf("%lld %lld %d %d", &e, &u, &a, &b) == 4) {
        const mj::DedupPlan p = mj::dedup_plan(e, u, a, b);
        printf("%d %d %d %d\n", p.bs, p.kb, p.bits, p.fits ? 1 : 0);
    }
}
"""
COUNTS = sorted({1, 2, 3, 4, 5, 8, 9, 10, 16, 17, 60, 1000, 65536, 65537, 300000, 1 << 20, 2 ** 31 - 1})
EXPECT = sorted({0, 1, 3071, 3072, 3073, 6144, 12287, 12289, 786432, 786433, 1300000, 1 << 24, 1 << 28,
                 1 << 31} | {3072 << b for b in range(16)} | {(3072 << b) + 1 for b in range(16)})


def key_bits(n):
    return max(n - 1, 0).bit_length()


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_bucket_bits_stay_within_the_keys(tmp_path):
    src = tmp_path / "plan.cpp"
    src.write_text(MAIN)
    exe = str(tmp_path / "plan")
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-I", CSRC, str(src), "-o", exe])
    cases = [(e, u, a, b) for e in EXPECT for u in {0, e // 9, e, 3 * e} for a in COUNTS for b in COUNTS]
    out = subprocess.run([exe], input="".join("%d %d %d %d\n" % c for c in cases), text=True,
                         capture_output=True, check=True).stdout.split()
    got = [tuple(map(int, out[i:i + 4])) for i in range(0, len(out), 4)]
    assert len(got) == len(cases)
    for (e, u, a, b), (bs, kb, bits, fits) in zip(cases, got):
        assert bs == key_bits(b) and kb == key_bits(a) + bs, (e, u, a, b)
        if fits:
            assert 0 <= bits <= min(kb, 14) and 0 <= kb - bits <= 31, (e, u, a, b, kb, bits)
    # what ordinary calls have fits; two strings with more candidates than their keys' buckets do not
    fit = {(e, a, b): g[3] for (e, u, a, b), g in zip(cases, got) if u == 0}
    # whether it fits does not depend on how many are different
    assert all(g[3] == fit[(e, a, b)] for (e, u, a, b), g in zip(cases, got))
    assert fit[(1300000, 300000, 300000)] and fit[(3072, 2, 2)] and fit[(6144, 60, 60)]
    assert not fit[(1300000, 9, 9)]
    assert not fit[(1 << 24, 2, 2)]
