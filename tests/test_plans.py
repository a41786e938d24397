"""Which kernel a call takes, and how (pq_measure_plan(): host arithmetic, no GPU): rules whose other side was measured to be slower."""
import pytest


@pytest.fixture(scope="module")
def plan(pqlib_path):
    from paper_2408_09992_amd import binding
    return binding.pq_measure_plan


@pytest.mark.parametrize("N,B,m,K", [(600_000, 52, 64, 1), (600_000, 52, 64, 100), (600_000, 200, 32, 10), (2_000_000, 200, 4, 1), (600_000, 200, 16, 1)])
def test_bounds_keep_the_compute_units_filled(plan, N, B, m, K):
    # fewer workgroups than compute units, so that floors can be shared, is slower: 600,000 items, m = 64, 52 queries, K = 1: 148 us with
    # 16 per query, 116 with 19
    p = plan("scan", N, B, m, 256, K)
    assert p["kernel"] == "bounds"
    tiles = -(-B // p["queries"])
    assert p["groups"] * tiles > 256 - tiles
