"""The on-chip count (a hash table per block) at the sizes where it can go wrong: items around
the table's slots and the largest item counted on chip, tables that overflow and are counted in
classes, merged neighbouring buckets, records of one and of many k-mers, 128-bit keys that
share a word, and counts at the 16-bit field's reach.  Bit-exact against the oracle."""
import numpy as np
import pytest

from tests.gpu_util import check

pytestmark = pytest.mark.gpu

SLOTS = {1: 4096, 2: 8192, 3: 2048}   # per 64-bit key table; half for 128-bit keys


def _kc():
    from paper_2407_07718_amd import kc
    return kc


def _reads(parts):
    offsets = np.zeros(len(parts) + 1, dtype=np.uint64)
    np.cumsum([len(p) for p in parts], out=offsets[1:])
    return (np.concatenate(parts) if parts else np.zeros(0, np.uint8)), offsets


def _random(rng, n):
    return np.frombuffer(b"ACGT", dtype=np.uint8)[rng.integers(0, 4, size=n)]


@pytest.mark.parametrize("variant", [1, 2, 3])
@pytest.mark.parametrize("k", [21, 31, 33, 63])
def test_distinct_keys_around_the_table(k, variant):
    """Two buckets of nearly all distinct k-mers, from half a table to beyond the largest
    item counted on chip (8 tables): the table overflows and is counted in classes."""
    rng = np.random.default_rng(100 + k + variant)
    slots = SLOTS[variant] // (1 if k <= 31 else 2)
    cfg = _kc().make_config(log2_buckets=1, small_variant=variant)
    for n in (slots, 2 * slots - 1, 2 * slots + 1, 5 * slots, 17 * slots):
        r = _random(rng, n + k - 1)
        check(r, np.array([0, len(r)], np.uint64), k, 11, 1, 1 << 20, 64, cfg, label=f"distinct {n}")


@pytest.mark.parametrize("k", [21, 31, 51])
@pytest.mark.parametrize("copies", [3, 40])
def test_merged_buckets(k, copies):
    """Many more buckets than blocks, so that a block counts neighbours together; then the
    same reads with their buckets counted alone."""
    rng = np.random.default_rng(7 * k + copies)
    genome = _random(rng, 600_000 // copies + 200)
    parts = [genome[s:s + 150] for s in rng.integers(0, len(genome) - 150, size=4000)] * (1 if copies > 3 else 2)
    r, off = _reads(parts)
    for lb in (14, 16, 18, 8):
        check(r, off, k, 15, 1, 1 << 20, 300, _kc().make_config(log2_buckets=lb), label=f"merged lb={lb}")


@pytest.mark.parametrize("k,m", [(2, 1), (3, 1), (5, 4), (12, 5), (31, 30), (31, 1), (32, 31), (63, 32), (63, 1)])
def test_record_shapes(k, m):
    """Records of one k-mer (m near k) and of as many as fit, for the smallest and largest k."""
    rng = np.random.default_rng(k * 64 + m)
    r, off = _reads([_random(rng, int(n)) for n in rng.integers(1, 400, size=300)])
    for lb in (0, 1, 3):
        check(r, off, k, m, 1, 1 << 20, 100, _kc().make_config(log2_buckets=lb), label=f"records m={m} lb={lb}")


@pytest.mark.parametrize("end", ["low", "high"])
def test_keys_sharing_a_word(end):
    """128-bit keys that agree in their low (high) word: 32 bases of suffix (19 of prefix)
    in common, thousands of them in one bucket, each seen several times."""
    rng = np.random.default_rng(5)
    fixed = np.frombuffer(b"A" * 19 + b"C" * 32, dtype=np.uint8).copy()
    fixed[rng.integers(0, 51, size=25)] = ord("G")
    parts = []
    for _ in range(3000):
        p = fixed.copy()
        if end == "low":
            p[1:19] = _random(rng, 18)
        else:
            p[19:] = _random(rng, 32)
        parts += [p] * int(rng.integers(1, 4))
    r, off = _reads(parts)
    for lb in (1, 6):
        check(r, off, 51, 21, 1, 1000, 64, _kc().make_config(log2_buckets=lb), label=f"shared {end} lb={lb}")


@pytest.mark.parametrize("k", [21, 51])
def test_counts_in_one_slot(k):
    """One k-mer seen 30,000 times beside others in one item: the 16-bit count, its pair's
    neighbour, and the largest item's boundary (32,768 k-mers at most in an item)."""
    rng = np.random.default_rng(k)
    unit = _random(rng, k)
    for n in (1, 2, 16_000, 30_000, 32_767, 32_768, 32_769, 70_000):
        parts = [unit] * n + [_random(rng, k) for _ in range(500)]
        r, off = _reads(parts)
        check(r, off, k, 11, 1, 1 << 20, 70_100, _kc().make_config(log2_buckets=1), label=f"one k-mer {n} times")
