"""Counts under budgets of one size to a fraction of the one-pass workspace: one pass with fewer
buckets, rounds with as many or fewer; the reads have few survivors, so each has to succeed.  The
bucket rule on both sides of its line.  A budgeted host call beside kept blocks of other calls.
Bit-exact against the oracle."""
import threading

import numpy as np
import pytest

import oracle
from paper_2407_07718_amd import kc
from tests.gpu_util import assert_same, check

pytestmark = pytest.mark.gpu

_ACGT = np.frombuffer(b"ACGT", np.uint8)


def _reads(seed, n, repeats=3):
    """n bases: a third in three copies, the reported k-mers a stretch of 2,000 more often."""
    rng = np.random.default_rng(seed)
    g = _ACGT[rng.integers(0, 4, size=n // repeats)]
    r = np.resize(g, n)
    r[-20_000:] = np.resize(g[:2000], 20_000)
    return r, np.array([0, n], np.uint64)


@pytest.mark.parametrize("k,options", [(21, {}), (31, {}), (31, dict(small_variant=2)), (51, {}), (51, dict(small_variant=3)),
                                       (31, dict(force_hbm=True)), (31, dict(log2_buckets=10))])
@pytest.mark.parametrize("n", [240_000, 400_000, 1_000_000])
def test_budgets(k, options, n):
    r, off = _reads(k + n, n)
    full = kc.kc_workspace_size(n, 1, k, kc.make_config(**options))
    ran = 0
    for part in (1.0, 0.995, 0.97, 0.9, 0.75, 0.6, 0.4):
        cfg = kc.make_config(hbm_budget=int(full * part), **options)
        if kc.kc_workspace_size(n, 1, k, cfg):
            check(r, off, k, 15, 5, 1 << 20, 64, cfg=cfg, label=f"budget {part}")
            ran += 1
    assert ran >= 4 or options.get("small_variant") == 2   # (rounds of its 131,072 k-mers at least)


@pytest.mark.parametrize("k,n,m8,m9", [(31, 240_000, 512, 128), (51, 240_000, 512, 256), (31, 500_000, 1024, 256),
                                       (31, 60_000, 128, 64), (21, 2_000_000, 1024, 1024)])
def test_bucket_rule(k, n, m8, m9):
    r, off = _reads(n, n)
    for m, buckets in ((8, m8), (9, m9), (15, m9)):
        got, _ = check(r, off, k, m, 2, 1 << 20, 64, label=f"m={m}")
        assert got.totals["buckets"] == buckets


def test_budget_beside_kept_blocks():
    sets = [_reads(i, n) for i, n in enumerate((30_000, 900_000, 400_000))]
    refs = [oracle.count(r, o, 31, 5, 1 << 20, 64) for r, o in sets]
    budget = int(kc.kc_workspace_size(400_000, 1, 31, None) * 0.75)
    bad = []

    def work(t):
        for i in range(9):
            j = (i + t) % 3
            try:
                cfg = kc.make_config(hbm_budget=budget) if j == 2 else None
                assert_same(kc.kc_count(*sets[j], 31, 15, 5, 1 << 20, 64, cfg), refs[j], f"set {j}")
            except Exception as e:   # noqa: BLE001 (reported by the main thread)
                bad.append(f"thread {t} set {j}: {e}")

    th = [threading.Thread(target=work, args=(t,)) for t in range(3)]
    [t.start() for t in th]
    [t.join() for t in th]
    assert not bad, bad[0]
