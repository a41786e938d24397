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


@pytest.mark.parametrize("N,B,m,K,shared", [
    (1_000_000, 40, 64, 10, 0), (1_500_000, 32, 64, 5, 0), (2_000_000, 56, 64, 20, 1), (1_509_979, 52, 64, 9, 1), (1_500_000, 250, 8, 1, 0), (4_000_000, 130, 4, 3, 0), (4_000_000, 200, 4, 10, 1),
    (700_000, 180, 16, 1, 0), (1_500_000, 130, 16, 10, 1), (200_000, 64, 64, 10, 0), (450_000, 64, 64, 100, 0), (300_000, 100, 64, 100, 1), (450_000, 160, 64, 1, 1)])
def test_floors_are_shared_where_that_pays(plan, N, B, m, K, shared):
    # m = 64, 1M items, 40 queries, K = 10: 162 us with shared floors, 147 without; 200,000, 64 queries 87 and 69
    p = plan("scan", N, B, m, 256, K)
    assert p["kernel"] == "bounds" and p["shared"] == shared


@pytest.mark.parametrize("N,B,K,fine", [(120_000, 1000, 3, 1), (120_000, 260, 12, 1), (120_000, 400, 60, 1), (500_000, 200, 6, 1), (1_500_000, 130, 12, 1), (500_000, 1000, 6, 1),
                                        (60_000, 400, 60, 0), (1_500_000, 400, 6, 0), (250_000, 130, 12, 0), (120_000, 260, 3, 0), (1_000_000, 300, 6, 0)])
def test_sixteen_bit_counts_where_they_pay(plan, N, B, K, fine):
    # m = 16.  120,000 items, 260 queries, K = 12: 53 us without them, 48 with; 60,000, 400, K = 60: 81 with, by pairs of queries 55
    p = plan("scan", N, B, 16, 256, K)
    assert p["fine"] == fine


@pytest.mark.parametrize("n,B,K,fine", [(200_000, 500, 10, 1), (200_000, 1000, 100, 1), (1_000_000, 200, 10, 1), (200_000, 64, 10, 0), (1_000_000, 64, 10, 0)])
def test_lists_have_sixteen_bit_counts_where_floors_are_shared(plan, n, B, K, fine):
    # m = 8.  1M candidates, 500 queries, K = 10: 210 us without, 184 with; not shared, 64 queries: 51 and 57
    p = plan("subset", n, B, 8, 256, K)
    assert p["fine"] == p["shared"] == fine


@pytest.mark.parametrize("N,B,K", [(600_000, 141, 500), (1_100_000, 300, 294)])
def test_floors_are_shared_by_two_queries_of_64_splits_too(plan, N, B, K):
    # 600,000 items, 141 queries, K = 500: 1258 us without, 731 with
    p = plan("scan", N, B, 64, 256, K)
    assert p["kernel"] == "bounds" and p["queries"] == 2 and p["shared"] == 1


@pytest.mark.parametrize("kind,N,B,m,K,groups", [("subset", 1_000_000, 300, 8, 100, 8), ("subset", 3_000_000, 305, 4, 200, 8), ("subset", 1_000_000, 180, 16, 100, 8),
                                                 ("subset", 1_000_000, 200, 8, 10, 16), ("scan", 142_000, 1013, 64, 82, 1), ("scan", 400_000, 1013, 64, 82, 1)])
def test_workgroups_that_share_floors_or_scan_everything_score_less(plan, kind, N, B, m, K, groups):
    # lists of 1M candidates, 300 queries, m = 8, K = 100: 331 us with 24 workgroups per query that do not share, 199 with 8 that do; 142,000 items of
    # 64 splits, 1013 queries, K = 82: 797 with two per query, 654 with one
    p = plan(kind, N, B, m, 256, K)
    assert p["kernel"] == "bounds" and p["groups"] == groups
    assert p["shared"] == (groups > 1)


@pytest.mark.parametrize("N,B,m,K,rounds", [(800_000, 300, 32, 10, 4), (1_500_000, 300, 32, 20, 4), (100_000, 400, 32, 10, 1), (500_000, 480, 16, 3, 2), (500_000, 480, 8, 10, 1)])
def test_samples_before_shared_floors(plan, N, B, m, K, rounds):
    # m = 32, 800,000 items, 300 queries, K = 10: 355 us with one round, 277 with four
    p = plan("scan", N, B, m, 256, K)
    assert p["kernel"] == "bounds" and p["shared"] == 1 and p["fine"] == 0 and p["rounds"] == rounds


@pytest.mark.parametrize("kind,N,B,m,K,pairs", [
    ("scan", 17_000, 600, 8, 150, 0), ("scan", 17_000, 900, 8, 150, 1), ("scan", 9000, 720, 16, 150, 0), ("scan", 5000, 600, 8, 2, 0), ("scan", 12_000, 650, 32, 100, 0),
    ("scan", 30_000, 800, 16, 100, 0), ("scan", 22_000, 800, 16, 10, 1), ("scan", 22_000, 530, 16, 100, 1), ("scan", 40_000, 450, 16, 5, 0), ("scan", 35_000, 600, 16, 2, 0),
    ("scan", 35_000, 600, 16, 20, 1), ("scan", 40_000, 800, 32, 10, 0), ("scan", 30_000, 450, 32, 5, 1), ("subset", 17_780, 652, 16, 1, 0), ("subset", 17_825, 162, 16, 10, 1),
    ("scan", 90_000, 250, 4, 130, 0), ("scan", 60_000, 430, 4, 100, 0), ("scan", 43_000, 340, 4, 100, 1), ("scan", 68_000, 158, 4, 182, 1), ("scan", 24_000, 1000, 4, 100, 0),
    ("scan", 16_000, 1000, 4, 40, 0), ("scan", 33_000, 170, 4, 40, 1)])
def test_two_queries_per_workgroup_where_that_pays(plan, kind, N, B, m, K, pairs):
    # m = 16, 40,000 items, 800 queries, K = 10: 86.8 us by pairs, 56 by bounds; 9000, 720, K = 150 37 and 27 by one workgroup per query; m = 4, 90,000, 250, K = 130 54 and 29
    assert (plan(kind, N, B, m, 256, K)["kernel"] in ("pairs", "list pairs")) == bool(pairs)


def test_lists_that_fill_their_last_round_well_enough(plan):
    # 59,869 candidates, 262 queries, m = 16, K = 118: 105 us by pairs, 127 by one query per workgroup
    assert plan("subset", 59_869, 262, 16, 256, 118)["kernel"] == "list pairs"


@pytest.mark.parametrize("N,B,m,b,K", [(1_000_000, 140, 4, 6000, 131), (1_000_000, 270, 16, 1500, 250)])
def test_floors_are_shared_beside_large_alphabets(plan, N, B, m, b, K):
    # four queries to a workgroup.  m = 16, b = 1500, 270 queries of 1M items, K = 250: 1359 us without shared floors, 837 with
    p = plan("scan16", N, B, m, b, K)
    assert p["kernel"] == "bounds" and p["queries"] == 4 and p["shared"] == 1


@pytest.mark.parametrize("N,B,m,b,K,pairs", [(35_673, 358, 4, 665, 146, 0), (25_444, 439, 8, 1492, 152, 0), (416_818, 253, 8, 604, 292, 0), (66_572, 426, 4, 1772, 4, 0),
                                             (136_065, 75, 8, 1444, 265, 1), (24_905, 467, 8, 588, 26, 1), (187_157, 157, 16, 296, 98, 1), (83_203, 172, 4, 1089, 6, 1),
                                             (90_000, 430, 4, 300, 100, 0), (43_000, 430, 4, 300, 40, 0), (43_000, 340, 4, 300, 40, 1)])
def test_two_queries_per_workgroup_with_two_byte_sub_ids(plan, N, B, m, b, K, pairs):
    # m = 8, b = 1492, 25,444 items, 439 queries, K = 152: 56 us by pairs, 38 without
    assert (plan("scan16", N, B, m, b, K)["kernel"] == "pairs") == bool(pairs)


@pytest.mark.parametrize("N,B,b,K,bits", [(321_782, 389, 300, 200, 16), (347_633, 170, 700, 171, 16), (350_000, 900, 1000, 100, 16), (928_212, 648, 304, 158, 8), (3_791_894, 128, 312, 413, 8), (1_000_000, 40, 1000, 100, 8),
                                          (1_000_000, 900, 300, 40, 8), (63_334, 598, 300, 31, 16), (55_795, 942, 300, 19, 16), (2_555_679, 252, 1000, 409, 8), (350_000, 390, 300, 10, 8), (1_000_000, 390, 1900, 200, 8), (1_000_000, 900, 1900, 400, 16)])
def test_sixteen_bit_fields_for_many_results_of_two_byte_sub_ids(plan, N, B, b, K, bits):
    # (bytes let so many items pass there that 321,782 items with 389 queries took the general kernel: 437 us and 193)
    p = plan("scan16", N, B, 16, b, K)
    assert (p["kernel"], p["field_bits"]) == ("bounds", bits)


@pytest.mark.parametrize("N,B,K,bounds", [(24_000, 1000, 40, 0), (32_500, 800, 58, 0), (33_000, 830, 40, 1), (24_000, 830, 20, 1)])
def test_rows_of_four_bytes_with_few_items_per_result(plan, N, B, K, bounds):
    # 24,000 items, 1000 queries, K = 40: 63 us by bounds, 37 by the short kernel
    assert (plan("scan", N, B, 4, 256, K)["kernel"] == "bounds") == bool(bounds)


@pytest.mark.parametrize("N,B,m,b,K,shared", [(2_000_000, 60, 8, 1500, 6, 0), (4_000_000, 100, 8, 1500, 6, 1), (2_000_000, 60, 8, 1500, 150, 1), (1_000_000, 100, 8, 1500, 6, 0),
                                              (1_000_000, 100, 8, 1500, 60, 1), (4_000_000, 60, 4, 4000, 6, 0)])
def test_two_byte_sub_ids_share_floors_between_many_workgroups(plan, N, B, m, b, K, shared):
    # (more than sixteen workgroups per query.)  m = 8, b = 1500, 60 queries of 2M items, K = 6: 57 us without shared floors, 72 with; K = 150 111 and 103
    p = plan("scan16", N, B, m, b, K)
    assert p["kernel"] == "bounds" and p["groups"] > 16 and p["shared"] == shared


@pytest.mark.parametrize("kind,N,B,m,b,K,groups", [("scan", 2_000_000, 110, 4, 256, 400, 16), ("scan16", 1_000_000, 110, 4, 1500, 250, 16), ("scan", 600_000, 100, 8, 256, 300, 16),
                                                   ("scan", 480_000, 110, 16, 256, 450, 16), ("scan", 650_000, 212, 8, 256, 30, 18), ("scan", 260_000, 98, 16, 256, 100, 19)])
def test_many_results_take_sixteen_workgroups_that_share_floors(plan, kind, N, B, m, b, K, groups):
    # m = 4, 2M items, 110 queries, K = 400: 163 us by eighteen workgroups that do not, 88 by sixteen
    p = plan(kind, N, B, m, b, K)
    assert (p["kernel"], p["groups"], p["shared"]) == ("bounds", groups, int(groups == 16))


@pytest.mark.parametrize("kind,N,B,m,b,K,shared", [("scan", 140_000, 169, 64, 256, 120, 1), ("scan", 70_000, 169, 64, 256, 30, 0), ("scan", 140_000, 125, 64, 256, 60, 0),
                                                   ("scan16", 340_000, 129, 4, 6000, 13, 0), ("scan16", 340_000, 129, 4, 6000, 30, 1), ("scan16", 700_000, 129, 4, 6000, 4, 0),
                                                   ("scan16", 700_000, 300, 4, 6000, 4, 1), ("scan16", 700_000, 60, 8, 3000, 30, 0), ("scan16", 700_000, 60, 8, 3000, 100, 1)])
def test_queries_of_one_word_share_floors_where_that_pays(plan, kind, N, B, m, b, K, shared):
    # m = 64, 170 queries of 140,000 items, K = 120: 292 us without shared floors, 208 with; m = 4, b = 6000, 129 of 700,000, K = 4 59 and 75
    p = plan(kind, N, B, m, b, K)
    assert p["kernel"] == "bounds" and p["shared"] == shared


@pytest.mark.parametrize("N,B,m,K", [(26_060, 3018, 8, 1), (102_314, 3141, 8, 2), (699_551, 2485, 8, 18), (3_670_000, 2800, 8, 1), (2_200_000, 2083, 8, 8), (298_538, 1563, 16, 2),
                                     (401_145, 1691, 16, 4), (85_607, 884, 32, 1), (868_457, 828, 32, 6), (300_000, 800, 8, 100)])
def test_static_scratch_holds_a_large_batchs_tables(plan, N, B, m, K):
    # without bounds 102,314 items, m = 8, 3141 queries, K = 2 take 416 us, with them 97
    assert plan("static", N, B, m, 256, K) == plan("scan", N, B, m, 256, K)
    assert plan("static", N, B, m, 256, K)["kernel"] == "bounds"


@pytest.mark.parametrize("N,B,m,K,instead", [(150_000, 8000, 8, 2, "pairs"), (400_000, 300, 64, 10, "pairs"), (1_000_000, 3000, 16, 100, "batched")])
def test_static_scratch_leaves_out_bounds_that_do_not_fit(plan, N, B, m, K, instead):
    assert plan("scan", N, B, m, 256, K)["kernel"] == "bounds"
    assert plan("static", N, B, m, 256, K)["kernel"] == instead


@pytest.mark.parametrize("N,B,m,K,queries", [
    (700_000, 17, 8, 10, 8), (5_000_000, 24, 8, 100, 8), (2_600_000, 20, 16, 128, 8), (10_000_000, 20, 16, 40, 8), (997_951, 17, 16, 128, 8), (443_030, 22, 16, 213, 8),
    (700_000, 33, 8, 10, 8), (3_500_000, 36, 8, 10, 8), (2_600_000, 33, 16, 102, 8), (3_000_000, 40, 16, 10, 8), (20_000_000, 36, 8, 200, 8), (9_000_000, 36, 16, 200, 8),
    (5_200_000, 36, 8, 200, 16), (9_000_000, 36, 8, 70, 16), (50_000_000, 40, 8, 10, 16), (10_000_000, 48, 8, 30, 16), (16_000_000, 33, 16, 10, 16),
    (1_300_000, 16, 8, 10, 16), (1_300_000, 25, 8, 10, 16), (1_300_000, 41, 8, 10, 16), (1_280_000, 64, 8, 10, 16)])
def test_eight_queries_per_workgroup_where_sixteen_leave_the_last_half_empty(plan, N, B, m, K, queries):
    # m = 8, 20 queries of 700,000 items, K = 10: 22.4 us by sixteens, 20.0 by eights; 36 queries of 5.2M, K = 200 88 and 100; 33 to 48 of long scans by pairs of lanes 98, by sixteens 90
    p = plan("scan", N, B, m, 256, K)
    assert (p["kernel"], p["queries"]) == ("bounds", queries)


@pytest.mark.parametrize("N,B,m,K,far", [
    (1_280_000, 64, 8, 10, 1), (1_280_000, 1024, 8, 100, 1), (180_003, 1000, 8, 6, 0), (137_321, 1650, 8, 100, 0), (5_000_000, 16, 16, 10, 2), (300_000, 64, 16, 20, 0),
    (80_000, 512, 8, 100, 0), (80_000, 1000, 8, 30, 0), (80_000, 512, 8, 10, 1), (100_000, 400, 8, 100, 1),
    (7_000_000, 48, 16, 200, 0), (12_000_000, 48, 16, 130, 0), (20_000_000, 80, 16, 100, 0), (12_000_000, 64, 16, 100, 2), (12_000_000, 32, 16, 130, 2), (12_000_000, 16, 16, 256, 2),
    (400_000, 600, 32, 4, 4), (50_000_000, 32, 8, 10, 2), (20_000_000, 32, 16, 10, 3), (1_280_000, 64, 4, 10, 0), (1_000_000, 8, 64, 10, 0)])
def test_splits_in_device_memory_and_the_room_for_their_rows(plan, N, B, m, K, far):
    # m = 8, 400,000 items, 512 queries, K = 6: 58.8 us with an eighth of the splits in device memory, 58.5 without; 64 of 1.28M, K = 10 32.0 and 32.6;
    # m = 16, 12M, 48, K = 200 375 and 343, 64, K = 100 0.97 as long with
    from paper_2408_09992_amd import binding
    p = plan("scan", N, B, m, 256, K)
    assert (p["kernel"], p["far"]) == ("bounds", far)
    tables = binding.pq_score_topk_workspace_bytes(N, B, m, 256, K) - 8 * K * B * p["groups"]
    a_query = 256 * m * (2 if p["field_bits"] == 16 else 1) + 512 + 16 + 256 * far
    others = 4 * p["parts"] * (K + 4) if p["parts"] > 1 else 0
    assert B * a_query <= tables <= -(-B // p["queries"]) * p["queries"] * (a_query + others) + 5 * 256


# One query by one-byte bounds or without.  Popular sub-ids (codes by Zipf(1.1)) gain less: m = 16, 6M, K = 10 23.7 us without and 24.4, K = 256 11M 47.3 and 49.4; m = 32, 3M 24.0 and 25.6,
# K = 256 8M 57.9 and 61.5; m = 64, 9M 104.0 and 107.8, 40M 429 and 424.  Two-byte sub-ids gain nothing while the last-level cache holds the codes (m = 8, b = 1024, 12.5M 38.3 and 39.7, 16M 46.6 and
# 48.7), larger alphabets at m = 16 nowhere (b = 800, 15M 88.7 and 89.6).
@pytest.mark.parametrize("kind,m,b,K,N,by_bytes", [("scan", 16, 256, 10, 6_000_000, False), ("scan", 16, 256, 10, 6_500_000, True), ("scan", 16, 256, 256, 11_000_000, False), ("scan", 16, 256, 256, 16_000_000, True),
                                                   ("scan", 32, 256, 10, 3_000_000, False), ("scan", 32, 256, 10, 4_500_000, True), ("scan", 32, 256, 256, 8_000_000, False), ("scan", 32, 256, 256, 10_100_000, True),
                                                   ("scan", 64, 256, 10, 9_000_000, False), ("scan", 64, 256, 100, 40_000_000, True), ("scan16", 8, 1024, 10, 12_500_000, False), ("scan16", 8, 1024, 10, 16_000_000, False),
                                                   ("scan16", 8, 1024, 10, 45_000_000, True), ("scan16", 4, 1500, 10, 14_000_000, False), ("scan16", 4, 1500, 10, 30_000_000, True), ("scan16", 16, 800, 10, 15_000_000, False),
                                                   ("scan16", 16, 300, 100, 4_000_000, False), ("scan16", 16, 300, 100, 5_000_000, True)])
def test_one_byte_bounds_where_they_pay(plan, kind, m, b, K, N, by_bytes):
    assert (plan(kind, N, 1, m, b, K)["field_bits"] == 8) == by_bytes


@pytest.mark.parametrize("N,B,m,K,rounds", [(8_500_000, 3, 8, 39, 1), (8_500_000, 3, 8, 217, 3), (4_400_000, 6, 8, 217, 2), (13_000_000, 2, 16, 39, 3), (8_500_000, 8, 16, 10, 1), (8_500_000, 16, 16, 10, 2), (24_000_000, 4, 4, 10, 1), (4_500_000, 40, 4, 217, 8), (24_000_000, 24, 4, 39, 5)])
def test_a_few_queries_samples_grow_by_parts_not_by_rounds(plan, N, B, m, K, rounds):
    # up to sixteen queries have sixteen parts with a compute unit each: 8.5M items, m = 8, 3 queries, K = 39 30.4 us with one round of these, 31.6 with two; more queries gain by larger
    # samples (24M, m = 4, 24, K = 39 80.1 with four, 75.4 with five)
    p = plan("scan", N, B, m, 256, K)
    assert p["kernel"] == "bounds" and p["rounds"] == rounds
