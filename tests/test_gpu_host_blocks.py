"""Memory that outlives a call: the device blocks of host calls (shared by threads, of growing and
shrinking sizes, and a call that fails) and a batch's results through pinned memory
(small and large sets, on their own and counted together, fetched again after a run on changed
reads).  Bit-exact against the oracle."""
import threading

import numpy as np
import pytest

import oracle
from paper_2407_07718_amd import synth
from tests.gpu_util import assert_same

pytestmark = pytest.mark.gpu


def _set(seed, n_reads):
    rng = np.random.Generator(np.random.PCG64(seed))
    g = synth.uniform_genome(rng, max(300, n_reads * 20))
    return synth.sample_reads(rng, g, rng.integers(30, 200, n_reads), p_sub=0.01, p_n=0.002)


def test_blocks_shared_by_threads():
    import torch
    from paper_2407_07718_amd import kc
    jobs = [(_set(i, n), k, m, b) for i, (n, k, m, b) in enumerate(
        [(3, 21, 11, 0), (5000, 31, 17, 0), (200, 51, 21, 0), (20000, 31, 17, 0), (1, 17, 9, 0), (9000, 31, 17, 40 << 20)])]
    refs = [oracle.count(r, o, k, 1, 100, 64) for (r, o), k, m, _ in jobs]
    bad = []

    def work(t):
        for i in range(12):
            j = (i * 5 + t) % len(jobs)
            (r, o), k, m, b = jobs[j]
            try:
                if b:   # (a budget whose survivor pool is too small for min_freq 1: refused)
                    with pytest.raises(kc.KCError):
                        kc.kc_count(r, o, k, m, 1, 100, 64, kc.make_config(hbm_budget=b))
                else:
                    assert_same(kc.kc_count(r, o, k, m, 1, 100, 64), refs[j], f"job {j}")
            except Exception as e:   # noqa: BLE001 (reported by the main thread)
                bad.append(f"thread {t} job {j}: {e}")

    free0 = torch.cuda.mem_get_info()[0]
    th = [threading.Thread(target=work, args=(t,)) for t in range(4)]
    [t.start() for t in th]
    [t.join() for t in th]
    assert not bad, bad[0]
    assert free0 - torch.cuda.mem_get_info()[0] < (4 << 30) + (1 << 29)


@pytest.mark.parametrize("sizes", [(40, 300, 5, 1, 90, 700), (60_000, 40, 50, 60), (50, 120_000)])
def test_batch_results_again(sizes):
    import torch
    from paper_2407_07718_amd import kc
    dev = torch.device("cuda:0")
    sets = [_set(100 + i, n) for i, n in enumerate(sizes)]
    k, m, lo, hi, H = 31, 17, 1, 1 << 20, 100
    d = [(torch.from_numpy(np.array(r)).to(dev), torch.from_numpy(np.array(o).view(np.int64)).to(dev)) for r, o in sets]
    b = kc.DeviceBatch([(r, o, k, m, lo, hi, H) for r, o in d])
    for turn in range(3):
        b.run()
        for again in range(2):
            for i, (r, o) in enumerate(sets):
                assert_same(b.result(i), oracle.count(r, o, k, lo, hi, H), f"turn {turn} set {i}")
        # the same lengths, other bases
        sets = [(np.roll(r, 7 + turn), o) for r, o in sets]
        for (t, _), (r, _) in zip(d, sets):
            t.copy_(torch.from_numpy(np.array(r)))
    b.close()
