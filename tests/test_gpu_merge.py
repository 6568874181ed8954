"""Merge of the large buckets' lists: as many entries as a block holds, fewer and more; lists of one
entry and long ones; keys of up to 32 bits and more (sorted as they are or mixed); a k-mer whose
entries alone are more than a block holds; several sets.  Bit-exact against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2407_07718_amd import kc
from tests.gpu_util import assert_same, check

pytestmark = pytest.mark.gpu

_ACGT = np.frombuffer(b"ACGT", dtype=np.uint8)


def _copies(rng, n, k, times):
    """n random k-mers, each as a read of its own, `times` over in another order each time."""
    r = _ACGT[rng.integers(0, 4, size=(n, k))]
    r = np.concatenate([r[rng.permutation(n)] for _ in range(times)])
    return r.reshape(-1), np.arange(n * times + 1, dtype=np.uint64) * k


@pytest.mark.parametrize("k", [13, 16, 17, 31, 32, 51])
@pytest.mark.parametrize("variant", [1, 3])
def test_entries(k, variant):
    """All k-mers of two buckets through the merge: about n / 2 distinct ones in each."""
    rng = np.random.default_rng(k * 4 + variant)
    cfg = kc.make_config(log2_buckets=1, force_hbm=True, small_variant=variant)
    for n, times in ((1, 1), (2, 3), (127, 9), (2000, 2), (8000, 1), (8192, 1), (8400, 2), (30_000, 3)):
        r, off = _copies(rng, n, k, times)
        check(r, off, k, 9, 1, 1 << 20, 64, cfg=cfg, label=f"{n} k-mers {times} times, variant {variant}")


@pytest.mark.parametrize("k", [31, 51])
def test_one_kmer_in_many_lists(k):
    """A stretch of one base: more lists with the one k-mer than entries a block holds."""
    rng = np.random.default_rng(k)
    n = 18_500_000 if k == 31 else 9_300_000
    r = np.concatenate([np.full(n, ord("A"), np.uint8), _ACGT[rng.integers(0, 4, 50_000)], np.full(3000, ord("T"), np.uint8)])
    got, _ = check(r, np.array([0, len(r)], np.uint64), k, 11, 1, 1 << 30, 64, cfg=kc.make_config(small_variant=3), label="one base")
    assert got.totals["list_entries"] > 4096 and got.totals["max_count"] >= n


def test_sets():
    """Several sets with large buckets counted together (the same k-mers in several of them)."""
    import torch
    rng = np.random.default_rng(5)
    sets = [_copies(rng, n, 31, 2) for n in (3000, 40, 9000)]
    sets.append(sets[0])
    d = [(torch.from_numpy(r).cuda(), torch.from_numpy(o.view(np.int64)).cuda()) for r, o in sets]
    b = kc.DeviceBatch([(r, o, 31, 9, 1, 1 << 20, 64) for r, o in d], kc.make_config(force_hbm=True))
    b.run()
    for i, (r, o) in enumerate(sets):
        assert_same(b.result(i), oracle.count(r, o, 31, 1, 1 << 20, 64), f"set {i}")
    b.close()
