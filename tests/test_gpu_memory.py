"""What host calls leave with the library goes back on request."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import assert_same

pytestmark = pytest.mark.gpu

_ACGT = np.frombuffer(b"ACGT", np.uint8)


def test_release_memory():
    import torch
    from paper_2407_07718_amd import kc
    rng = np.random.default_rng(1)
    r = _ACGT[rng.integers(0, 4, size=2_000_000)]
    off = np.array([0, len(r)], np.uint64)
    ref = oracle.count(r, off, 31, 1, 1 << 20, 64)
    kc.kc_count(r, off, 31, 17, 1, 1 << 20, 64)   # (the first launch loads the library's own buffers)
    kc.kc_release_memory()
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    for _ in range(2):
        assert_same(kc.kc_count(r, off, 31, 17, 1, 1 << 20, 64), ref)
        held = free - torch.cuda.mem_get_info()[0]
        assert held > 60 * len(r)
        assert held >= kc.kc_release_memory() > 60 * len(r)
        assert free - torch.cuda.mem_get_info()[0] < 8 << 20
    assert kc.kc_release_memory() == 0
