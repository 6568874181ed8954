"""The extension version's two one-pass ways (all windows sorted; the pairs counted and the
windows looked up in them) on both sides of where the choice changes: base counts around 2^22
and 2^25, min_freq 1 and 2, k around 29 and around the key widths, values that hold (read,
position) and values that hold a base offset, heavy k-mers, capacities cut short, and a
workspace that only the sort fits.  Bit-exact against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2407_07718_amd import synth
from tests.test_gpu_ext import assert_same_ext, check_ext

pytestmark = pytest.mark.gpu

N = 1 << 22


def _reads(seed, bases, long_read=0):
    """Reads of 100 to 300 bases (behind one of `long_read`) with errors and N, `bases` in all,
    over a genome that they cover about five times, a poly-A stretch in it."""
    rng = np.random.Generator(np.random.PCG64(seed))
    g = synth.uniform_genome(rng, bases // 5)
    g[1000:1200] = g[1000]
    lens = rng.integers(100, 301, bases // 100)
    if long_read:
        lens = np.concatenate([[long_read], lens])
    ends = np.minimum(np.cumsum(lens), bases)
    lens = np.diff(np.concatenate([[0], ends[: np.searchsorted(ends, bases) + 1]]))
    body = synth.sample_reads(rng, g, lens[1:] if long_read else lens, p_sub=0.005, p_n=0.001)
    reads, off = body
    if long_read:
        reads = np.concatenate([np.resize(g, long_read), reads])
        off = np.concatenate([[0], off + np.uint64(long_read)]).astype(np.uint64)
    assert len(reads) == bases
    return reads, off


@pytest.mark.parametrize("bases,k,lo,long_read", [
    (N - 1, 32, 2, 0), (N, 32, 2, 0), (N + 4095, 51, 1, 0), (N + 17, 33, 3, 0), (N, 63, 2, 0),
    (N + 5, 51, 2, N // 2 + 1), (N + 1, 31, 2, 0), (8 * N - 1, 31, 2, 0), (8 * N, 31, 2, 0), (8 * N + 33, 29, 2, 0),
    (8 * N, 28, 2, 0), (8 * N + 5, 30, 2, N)])
def test_ext_count(bases, k, lo, long_read):
    reads, off = _reads(bases + k, bases, long_read)
    check_ext(reads, off, k, lo, 1 << 20, 200, label=f"{bases} bases")


@pytest.mark.parametrize("short", [True, False])
def test_ext_count_limits(short):
    """Capacities below the result: the parts that fit, and the totals; a workspace that only
    the sort of all windows fits: the same result."""
    import torch
    from paper_2407_07718_amd import kc
    reads, off = _reads(3, N, 0)
    ref = oracle.count_ext(reads, off, 33, 2, 50, 64)
    n, n_occ = ref.base.n_pairs, int(ref.occ_off[-1])
    pc, oc = (n // 3, n_occ // 3) if short else (n, n_occ)
    ctr = kc.DeviceExtCounter(len(reads), len(off) - 1, 33, 2, 50, 64, pair_capacity=pc, occ_capacity=oc)
    if not short:
        ctr.workspace = ctr.workspace[: 47 * len(reads) + (8 << 20)]
    d_r = torch.from_numpy(reads).cuda()
    d_o = torch.from_numpy(off.view(np.int64)).cuda()
    if short:
        with pytest.raises(kc.KCError):
            ctr.count(d_r, d_o)
        assert np.array_equal(ctr.counts[:pc].cpu().numpy().view(np.uint32), ref.base.counts[:pc])
        assert np.array_equal(ctr.occ_off[:pc].cpu().numpy().view(np.uint64), ref.occ_off[:pc])
        assert np.array_equal(ctr.occ_read[:oc].cpu().numpy().view(np.uint32), ref.occ_read[:oc])
        assert np.array_equal(ctr.occ_pos[:oc].cpu().numpy().view(np.uint32), ref.occ_pos[:oc])
    else:
        assert_same_ext(ctr.result(ctr.count(d_r, d_o)), ref, "sorted in a smaller workspace")
