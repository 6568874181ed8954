"""Prefix sums of the partition and of the bucket plan: arrays that end inside a group of four, a
row, a wave's and a block's share, by one block and by many, and one or several blocks of buckets.
Bit-exact against the oracle."""
import numpy as np
import pytest

from paper_2407_07718_amd import kc
from tests.gpu_util import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("log2b", [1, 2, 3, 9, 10, 11, 13, 20])
def test_scan_lengths(log2b):
    rng = np.random.default_rng(log2b)
    for n in (60, 1500, 5000, 17_000, 40_001, 300_000, 1_300_000):
        r = np.frombuffer(b"ACGT", np.uint8)[rng.integers(0, 4, size=n)]
        r[rng.integers(0, n, n // 400)] = ord("N")
        cuts = np.unique(np.concatenate([[0, n], rng.integers(0, n, n // 300)])).astype(np.uint64)
        check(r, cuts, 25, 9, 1, 1 << 20, 64, cfg=kc.make_config(log2_buckets=log2b), label=f"2^{log2b} buckets")
