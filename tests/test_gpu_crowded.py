"""Survivors whose keys share their leading 32 bits: groups of k-mers with 17 bases in common, of the
lengths where the ranking of a bin gives way to radix passes, in ranges that one wave and one block
sort, for 64- and 128-bit keys, and for several sets sorted in place.  Bit-exact against the oracle."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import assert_same, check

pytestmark = pytest.mark.gpu

_ACGT = np.frombuffer(b"ACGT", dtype=np.uint8)


def _groups(rng, k, sizes, others):
    """Reads of one k-mer each: groups that share their first 17 bases, and unrelated ones."""
    n = sum(sizes) + others
    r = rng.integers(0, 4, size=(n, k), dtype=np.uint8)
    at = 0
    for s in sizes:
        p = rng.integers(0, 4, size=17, dtype=np.uint8)
        p[0] = 0
        r[at:at + s, :17] = p
        r[at:at + s, -1] = 1      # (its reverse complement starts with G)
        at += s
    return _ACGT[rng.permutation(r)].reshape(-1), np.arange(n + 1, dtype=np.uint64) * k


@pytest.mark.parametrize("k", [31, 51])
def test_crowded_bins(k):
    rng = np.random.default_rng(k)
    for sizes, others in (([64], 3000), ([65], 3000), ([66] * 9, 200_000), ([300, 447, 448, 449, 64, 65], 150_000),
                          ([767, 768, 769], 100_000), ([1500, 2047, 2048, 2049], 100_000),
                          ([4000, 4095, 4096, 4097, 65], 100_000), ([9000], 50_000)):
        r, off = _groups(rng, k, sizes, others)
        check(r, off, k, 15, 1, 1 << 20, 64, label=f"groups of {sizes} among {others}")


@pytest.mark.parametrize("hi", [1000, (1 << 32) - 1])
def test_crowded_bins_of_sets(hi):
    from paper_2407_07718_amd import kc
    rng = np.random.default_rng(9)
    for k in (31, 51):
        jobs = [kc.Job(*_groups(rng, k, sizes, 40_000), k, 15, 1, hi, 64)
                for sizes in ([70, 300], [700, 500, 449], [2048, 3000], [5000])]
        for i, (got, j) in enumerate(zip(kc.kc_count_batch(jobs), jobs)):
            assert_same(got, oracle.count(j.reads, j.offsets, k, 1, hi, 64), f"k={k} set {i}")
