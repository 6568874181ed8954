"""Buckets of many distinct k-mers: counted by their block in two classes, left to the second launch
in four to 16, or cut into chunks, at the sizes where they change hands; several at a time per block,
one per block, in rounds and for several sets; unique k-mers and k-mers of some copies; all three
kinds in one count.  Every figure bit-exact against the oracle."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import assert_same, check

pytestmark = pytest.mark.gpu

_ACGT = np.frombuffer(b"ACGT", dtype=np.uint8)


def _reads(rng, n, copies, sub=0.0):
    r = np.resize(_ACGT[rng.integers(0, 4, size=max(70, n // copies))], n)
    if sub:
        e = rng.random(n) < sub
        r = np.where(e, _ACGT[rng.integers(0, 4, size=n)], r)
    return r, np.array([0, n], np.uint64)


# slots of a table (k = 21 and 31: 4,096, 8,192, 2,048; k = 51: half), tables per bucket
@pytest.mark.parametrize("k", [21, 31, 51])
@pytest.mark.parametrize("variant,slots", [(1, 4096), (2, 8192), (3, 2048)])
@pytest.mark.parametrize("tables", [0.9, 1.0, 1.1, 1.6, 2.4, 4, 7.5, 8.5])
def test_tables_per_bucket(k, variant, slots, tables):
    from paper_2407_07718_amd import kc
    rng = np.random.default_rng(int(100 * tables) + k)
    slots //= 1 if k <= 31 else 2
    for copies, sub in ((1, 0.0), (3, 0.01), (40, 0.0)):
        r, off = _reads(rng, int(tables * slots * 16), copies, sub)
        cfg = kc.make_config(log2_buckets=4, small_variant=variant)
        check(r, off, k, 13, 1 if copies == 1 else 2, 1 << 20, 64, cfg=cfg, label=f"{tables} tables, {copies} copies")


@pytest.mark.parametrize("k,m", [(15, 5), (21, 6), (31, 5), (51, 6), (51, 7)])
@pytest.mark.parametrize("copies", [1, 5])
def test_small_minimizers(k, m, copies):
    """Chunks, classes and buckets of one block in one count."""
    rng = np.random.default_rng(k + m)
    for n in (200_000, 1_000_000, 5_000_000):
        r, off = _reads(rng, n, copies, 0.002)
        check(r, off, k, m, 1, 1 << 20, 64, label=f"{copies} copies")


@pytest.mark.parametrize("k", [21, 51])
def test_rounds(k):
    from paper_2407_07718_amd import kc
    rng = np.random.default_rng(k)
    n = 3_000_000
    r, off = _reads(rng, n, 4, 0.01)
    full = kc.kc_workspace_size(n, 1, k, None)
    for m in (6, 15):
        check(r, off, k, m, 3, 1 << 20, 64, cfg=kc.make_config(hbm_budget=int(full * 0.7)), label="rounds")


@pytest.mark.parametrize("hi", [1000, (1 << 32) - 1])
def test_sets(hi):
    from paper_2407_07718_amd import kc
    rng = np.random.default_rng(8)
    for k, m in ((21, 5), (51, 6)):
        jobs = [kc.Job(*_reads(rng, n, c, 0.005), k, m, 1, hi, 64)
                for n, c in ((300_000, 1), (5_000, 1), (800_000, 6), (120_000, 2), (64_000, 1))]
        for i, (got, j) in enumerate(zip(kc.kc_count_batch(jobs), jobs)):
            assert_same(got, oracle.count(j.reads, j.offsets, k, 1, hi, 64), f"k={k} set {i}")


def test_replays_of_a_graph():
    """The list of buckets left over starts empty in every replay."""
    import torch
    from paper_2407_07718_amd import kc
    rng = np.random.default_rng(2)
    r, off = _reads(rng, 1_000_000, 2, 0.01)
    d = torch.from_numpy(r).cuda()
    o = torch.from_numpy(off.view(np.int64)).cuda()
    ctr = kc.DeviceCounter(len(r), 1, 21, 6, 1, 1 << 20, 64)
    ctr.count(d, o)
    st = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        ctr.count(d, o, sync=False)
    for turn in range(4):
        r2, _ = _reads(rng, 1_000_000, 1 + turn, 0.01)
        d.copy_(torch.from_numpy(r2))
        g.replay()
        torch.cuda.synchronize()
        tot = kc.kc_totals.from_buffer_copy(ctr.totals.cpu().numpy().tobytes()).as_dict()
        assert_same(ctr.result(tot), oracle.count(r2, off, 21, 1, 1 << 20, 64), f"replay {turn}")
        (torch.ones(1000, device="cuda") * turn).sum().item()
