"""The survivors' coarse pass from where the count left them: segments of none, one row, a row and
one, many rows; fewer segments than waves and many more; and survivors of merged runs next to
buckets' or alone.  Bit-exact against the oracle."""
import numpy as np
import pytest

from paper_2407_07718_amd import kc
from tests.gpu_util import check

pytestmark = pytest.mark.gpu

_ACGT = np.frombuffer(b"ACGT", dtype=np.uint8)


def _reads(rng, n, k):
    """n reads of k + 1 bases, twice each."""
    r = _ACGT[rng.integers(0, 4, size=(n, k + 1))]
    return np.concatenate([r, r]).reshape(-1), np.arange(2 * n + 1, dtype=np.uint64) * (k + 1)


@pytest.mark.parametrize("k", [21, 31, 40])
@pytest.mark.parametrize("log2b", [1, 5, 9, 12, 18])
def test_segments(k, log2b):
    rng = np.random.default_rng(k * 32 + log2b)
    for n in (1, 31, 32, 33, 64, 65, 3000, 70_000):
        r, off = _reads(rng, n, k)
        check(r, off, k, 11, 2, 100, 64, cfg=kc.make_config(log2_buckets=log2b), label=f"{n} reads, 2^{log2b} buckets")


@pytest.mark.parametrize("k,m", [(21, 2), (31, 1), (51, 3)])
@pytest.mark.parametrize("force", [0, 1])
def test_runs_and_buckets(k, m, force):
    """Few distinct minimizers: large buckets (merged runs) next to on-chip ones; all large."""
    rng = np.random.default_rng(k + force)
    for n in (40, 5000, 120_000):
        r, off = _reads(rng, n, k)
        check(r, off, k, m, 2, 100, 64, cfg=kc.make_config(log2_buckets=6, force_hbm=force), label=f"{n} reads, m={m}")
