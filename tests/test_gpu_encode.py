"""Encoding of the reads: every byte value in every place of a 32-byte word, either case, runs of
non-bases, and ends around multiples of 32 and of 64 threads' words.  Bit-exact against the
oracle."""
import numpy as np
import pytest

from tests.gpu_util import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [3, 8, 21])
def test_all_bytes(k):
    """Byte v once at each place of a word, bases around it."""
    rng = np.random.default_rng(k)
    r = np.frombuffer(b"ACGTacgt", np.uint8)[rng.integers(0, 8, size=256 * 32 * 64)]
    r[np.arange(256 * 32) * 64 + np.tile(np.arange(32), 256)] = np.repeat(np.arange(256), 32).astype(np.uint8)
    check(r, np.array([0, len(r)], np.uint64), k, 2, 1, 1 << 20, 64, label="all bytes")


@pytest.mark.parametrize("n", [1, 31, 32, 33, 2047, 2048, 2049, 16_385, 70_001])
def test_ends(n):
    rng = np.random.default_rng(n)
    r = rng.choice(np.frombuffer(b"ACGTacgtNn.-\x00\xff", np.uint8), size=n, p=[0.12] * 8 + [0.04 / 6] * 6)
    cuts = np.unique(np.concatenate([[0, n], rng.integers(0, n + 1, n // 500)])).astype(np.uint64)
    check(r, cuts, 15, 7, 1, 1 << 20, 64, label="ends")
