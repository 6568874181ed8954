"""The bucket rule on both sides of its lines: k-mer counts around 64 buckets of 512 and of half a
table, minimizers of 8 and 9 bases, the workspace of one size for both, budgets that make rounds.
Bit-exact against the oracle."""
import numpy as np
import pytest

from paper_2407_07718_amd import kc
from tests.gpu_util import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [17, 31, 32, 51])
@pytest.mark.parametrize("m", [8, 9])
def test_rule(k, m):
    rng = np.random.default_rng(k * 16 + m)
    for n in (32_767, 32_769, 65_537, 131_071, 131_073, 262_145, 524_289, 2_097_153):
        g = np.frombuffer(b"ACGT", np.uint8)[rng.integers(0, 4, size=n // 3)]
        r = np.concatenate([g, g, g])[:n]
        got, _ = check(r, np.array([0, len(r)], np.uint64), k, m, 1, 1 << 20, 64, label=f"{n} bases, m={m}")
        assert got.totals["buckets"] >= 64 or n < 65_536


@pytest.mark.parametrize("k", [31, 51])
def test_rule_and_budget(k):
    rng = np.random.default_rng(k)
    n = 400_000
    r = np.resize(np.frombuffer(b"ACGT", np.uint8)[rng.integers(0, 4, size=n // 3)], n)
    off = np.array([0, n], np.uint64)
    full = kc.kc_workspace_size(n, 1, k, None)
    for part in (0.3, 0.6, 0.99):
        cfg = kc.make_config(hbm_budget=int(full * part))
        if not kc.kc_workspace_size(n, 1, k, cfg):
            continue
        try:
            check(r, off, k, 9, 2, 1 << 20, 64, cfg=cfg, label=f"budget {part}")
        except kc.KCError as e:   # (the smaller budgets' pools hold fewer pairs than these reads have)
            assert part < 0.99 and "pool" in str(e)
