"""Several read sets counted together with no upper frequency bound: the survivors are sorted as
wide keys (set << 2k | k-mer), at k-mers of a few bits too, with many and few sets.  Bit-exact
against the oracle."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import assert_same

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [2, 3, 8, 14, 15, 16, 17, 31, 32])
@pytest.mark.parametrize("sizes", [(4000, 1, 90_000), tuple(range(700, 9100, 210)), (400_000, 300_000)])
def test_sets_of_short_keys(k, sizes):
    from paper_2407_07718_amd import kc
    rng = np.random.default_rng(k * 100 + len(sizes))
    jobs = []
    for n in sizes:
        r = np.frombuffer(b"ACGT", np.uint8)[rng.integers(0, 4, size=n)]
        jobs.append(kc.Job(r, np.unique(np.append(np.arange(0, n, 997), n)).astype(np.uint64), k, max(1, k // 2), 1,
                           (1 << 32) - 1, 64))
    print(f"case wide keys: k={k}, {len(jobs)} sets", flush=True)
    for i, (got, j) in enumerate(zip(kc.kc_count_batch(jobs), jobs)):
        assert_same(got, oracle.count(j.reads, j.offsets, k, 1, (1 << 32) - 1, 64), f"set {i}")
