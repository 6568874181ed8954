"""Memory budgets that the counts were accepted with when the workspace was last sized by its parts:
the smallest of them for inputs of every size and option that they depend on.  A budget that was
enough stays enough, whatever the regions are now, and the plan stays within it."""
import pytest

# bases, reads, k, options, bytes
SMALLEST = [
    (0, 1, 31, dict(), 1687958),
    (100, 1, 63, dict(), 1778160),
    (5000, 33, 21, dict(), 1930376),
    (60000, 400, 31, dict(), 4677184),
    (60000, 400, 32, dict(small_variant=3), 5209865),
    (100000, 666, 17, dict(), 5985854),
    (100000, 666, 51, dict(small_variant=3), 6327160),
    (240000, 1600, 31, dict(), 8702322),
    (240000, 1600, 31, dict(small_variant=2), 13922388),
    (240000, 1600, 51, dict(), 14206622),
    (240000, 1600, 17, dict(force_hbm=1), 8509130),
    (300000, 2000, 21, dict(), 9380172),
    (300000, 2000, 31, dict(small_variant=1), 12175864),
    (300000, 2000, 63, dict(small_variant=3), 14486767),
    (500000, 3333, 31, dict(), 19212510),
    (1000000, 6666, 51, dict(small_variant=3), 30658649),
    (1000000, 6666, 21, dict(log2_buckets=10), 31110058),
    (5300000, 35333, 31, dict(), 33504592),
    (10000000, 66666, 63, dict(), 38362413),
    (10000000, 66666, 32, dict(small_variant=3), 36266367),
    (100000000, 666666, 31, dict(), 91084226),
    (1000000000, 6666666, 31, dict(), 618894849),
    (1000000000, 6666666, 51, dict(log2_buckets=20), 620434186),
]


@pytest.mark.parametrize("bases,reads,k,options,budget", SMALLEST)
def test_smallest_budgets_stay_enough(bases, reads, k, options, budget):
    from paper_2407_07718_amd import kc
    size = kc.kc_workspace_size(bases, reads, k, kc.make_config(hbm_budget=budget, **options))
    assert 0 < size <= budget
