"""The survivors' sort reads them from the buckets' k-mer slots in equal shares: one bucket of most
k-mers, buckets that blocks count several at a time (whose survivors lie at the first ones' slots),
empty buckets, more buckets than k-mers, inputs of a row, a block's share and one more.  Every k-mer
reported or few of them.  Bit-exact against the oracle."""
import numpy as np
import pytest

from tests.gpu_util import check

pytestmark = pytest.mark.gpu

_ACGT = np.frombuffer(b"ACGT", dtype=np.uint8)


@pytest.mark.parametrize("k,m", [(21, 1), (31, 11), (51, 2), (51, 21)])
@pytest.mark.parametrize("log2_buckets", [0, 1, 6, 13, 16, 19])
def test_slots(k, m, log2_buckets):
    from paper_2407_07718_amd import kc
    rng = np.random.default_rng(k + 100 * log2_buckets)
    for n, copies in ((k, 1), (k + 63, 1), (k + 64, 1), (16_384 + k - 1, 1), (16_384 + k, 2), (70_001, 5), (900_007, 1),
                      (900_007, 3)):
        if m < 3 and n > 100_000:   # (one block would merge them all)
            n = 120_001
        r = np.resize(_ACGT[rng.integers(0, 4, size=max(k, n // copies))], n)
        for lo in (1, 2):
            check(r, np.array([0, n], np.uint64), k, m, lo, 1 << 20, 64, cfg=kc.make_config(log2_buckets=log2_buckets),
                  label=f"2^{log2_buckets} buckets, {copies} copies")


def test_several_buckets_at_a_time():
    """8 buckets and more per block, of very unequal sizes: poly-A and repeats beside unique bases."""
    from paper_2407_07718_amd import kc
    rng = np.random.default_rng(4)
    u = _ACGT[rng.integers(0, 4, size=3_000_000)]
    rep = np.tile(_ACGT[rng.integers(0, 4, size=173)], 3000)
    r = np.concatenate([u, rep, np.full(200_000, ord("A"), np.uint8), u[:500_000], rep])
    off = np.array([0, len(u), len(u) + len(rep), len(r)], np.uint64)
    for k, log2_buckets in ((21, 14), (31, 16), (51, 14), (51, 18)):
        for lo in (1, 2):
            check(r, off, k, 13, lo, 1 << 30, 64, cfg=kc.make_config(log2_buckets=log2_buckets), label="unequal buckets")


@pytest.mark.parametrize("k,m", [(21, 13), (51, 21)])
@pytest.mark.parametrize("log2_buckets", [12, 13, 14, 15])
def test_waves_that_share_buckets(k, m, log2_buckets):
    """19 shares of 3 to 27 times 64 buckets: rows dealt to all waves of a block, to half of them, ... to one;
    a long repeat makes one bucket of many rows among them."""
    from paper_2407_07718_amd import kc
    rng = np.random.default_rng(log2_buckets)
    u = _ACGT[rng.integers(0, 4, size=280_017)]
    r = np.concatenate([u, np.tile(u[:300], 60), u[1000:3000]])
    for lo in (1, 2):
        check(r, np.array([0, len(r)], np.uint64), k, m, lo, 1 << 20, 64,
              cfg=kc.make_config(log2_buckets=log2_buckets), label="shared buckets")
