"""The survivors' sort by key ranges at the lengths where a range changes hands (one wave, one
block, passes through HBM), with keys spread over the ranges and with keys that fall into one
range and one bin.  Bit-exact against the oracle."""
import numpy as np
import pytest

from tests.gpu_util import check

pytestmark = pytest.mark.gpu

_ACGT = np.frombuffer(b"ACGT", dtype=np.uint8)


def _kmers(rng, n, k, prefix):
    """n reads of one k-mer each; with `prefix` bases of poly-A in front (so that the read is
    its own canonical form and all keys share their leading bits)."""
    r = _ACGT[rng.integers(0, 4, size=(n, k))]
    if prefix:
        r[:, :prefix] = ord("A")
        r[:, -1] = ord("C")       # (the reverse complement starts with G)
    return r.reshape(-1), np.arange(n + 1, dtype=np.uint64) * k


@pytest.mark.parametrize("k", [21, 31, 51])
@pytest.mark.parametrize("prefix", [0, 8, 17])
def test_range_lengths(k, prefix):
    rng = np.random.default_rng(k * 100 + prefix)
    for n in (1, 2, 64, 65, 447, 448, 449, 512, 513, 767, 768, 769, 2047, 2048, 2049, 4095, 4096, 4097, 9001):
        if prefix and 4 ** (k - 1 - prefix) < n:
            continue
        r, off = _kmers(rng, n, k, prefix)
        check(r, off, k, 11, 1, 1 << 20, 64, label=f"{n} keys, {prefix} bases in common")


@pytest.mark.parametrize("k", [2, 3, 8, 15, 16, 17, 32, 33])
def test_short_keys(k):
    """Keys of fewer bits than a place has, and 128-bit keys with an empty high word."""
    rng = np.random.default_rng(k)
    r = _ACGT[rng.integers(0, 4, size=200_000)]
    check(r, np.array([0, len(r)], np.uint64), k, max(1, k // 2), 1, 1 << 20, 64, label="short keys")
