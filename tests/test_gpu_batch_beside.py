"""A batch's results read by one thread while another runs the batch again on changed reads: what
is read after the run is the run's.  Bit-exact against the oracle."""
import threading

import numpy as np
import pytest

import oracle
from paper_2407_07718_amd import synth
from tests.gpu_util import assert_same

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hi", [1 << 20, (1 << 32) - 1])   # (count and set in one value; as wide keys)
def test_result_during_run(hi):
    import torch
    from paper_2407_07718_amd import kc
    dev = torch.device("cuda:0")
    k, m, lo, H, n = 31, 17, 2, 64, 4_000_000
    rng = np.random.Generator(np.random.PCG64(11))
    off = np.arange(0, n + 1, 200, dtype=np.uint64)

    def reads(genome):
        g = synth.uniform_genome(rng, genome)
        start = rng.integers(0, genome - 200, len(off) - 1)
        return np.frombuffer(b"ACGT", np.uint8)[g[(start[:, None] + np.arange(200)).reshape(-1)]]

    # every turn has other numbers of pairs
    turns = [[reads(genome + 1000 * i) for i in range(3)] for genome in (400_000, 150_000, 300_000, 90_000)]
    d = [torch.from_numpy(r).to(dev) for r in turns[0]]
    d_off = torch.from_numpy(off.view(np.int64)).to(dev)
    b = kc.DeviceBatch([(r, d_off, k, m, lo, hi, H) for r in d])
    assert b.info()["shared"] == 3
    st = torch.cuda.Stream()   # (does not wait for the copies of the other thread)
    b.run(st)
    for turn, sets in enumerate(turns):
        for t, r in zip(d, sets):
            t.copy_(torch.from_numpy(r))
        torch.cuda.synchronize()
        stop = threading.Event()

        def reader():
            while not stop.is_set():
                try:
                    b.result(0)   # (the last run's, this one's, or neither's)
                except kc.KCError:
                    pass

        th = threading.Thread(target=reader)
        th.start()
        try:
            for _ in range(5):
                b.run(st)
        finally:
            stop.set()
            th.join()
        for i, r in enumerate(sets):
            assert_same(b.result(i), oracle.count(r, off, k, lo, hi, H), f"turn {turn} set {i}")
    b.close()
