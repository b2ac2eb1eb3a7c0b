"""The rules that choose a path or a launch by sizes, built for the host (tests/host/rules.cpp)."""
import pytest

RESIDENT = 1024  # sweep workgroups the chip holds: 256 compute units, four each


@pytest.mark.parametrize("f16", [0, 1])
def test_long_tile_groups_leave_enough_workgroups(rules, f16):
    """Groups above four tiles only where the launch still has many rounds of resident workgroups: a map of one
    strip and 1,500 tiles would otherwise leave compute units idle, one of 6,000 tiles half of them."""
    for M in (1, 256, 512, 513, 1024, 4096, 16384, 65025, 1 << 20):
        strips = rules.strips(M, 8)
        for nt in (1, 2, 187, 1499, 1500, 3000, 5999, 6000, 12000, 12500, 19999, 20000, 30000, 31250, 62500, 125000,
                   250000, 1 << 28):
            g = rules.group_tiles(nt, strips, 8, f16)
            assert g % 4 == 0 and 4 <= g <= 32
            assert g == 4 or -(-nt // g) * strips >= 8 * RESIDENT, (M, nt, g)


def test_tile_groups_of_many_strips_are_long(rules):
    assert rules.group_tiles(62500, 2048, 8, 0) == 8 and rules.group_tiles(62500, 2048, 8, 1) == 32
    assert rules.group_tiles(2000, 2048, 8, 1) == 8 and rules.group_tiles(31250, 8, 8, 0) == 8


@pytest.mark.parametrize("f16", [0, 1])
def test_searches_without_a_plan_end_where_long_rows_are_shared(rules, f16):
    """Few rows of a dozen ids are searched without a plan; rows of hundreds of ids on a large map, whose codebook
    rows a plan reads once per tile instead of once per sample, are not (at 1,000 ids each: 64 rows on 512 x 512)."""
    def direct(N, M, ids, ta=8):
        return rules.rows_direct(N, M, N * ids, ta, f16)

    for N, M in ((1, 4096), (33, 65536), (64, 1 << 18), (16, 1 << 20), (256, 65536), (1024, 4096), (4096, 256)):
        assert direct(N, M, 12), (N, M)
    for N, M in ((64, 1 << 18), (48, 1 << 18), (16, 1 << 20), (256, 65536)):
        assert not direct(N, M, 1000), (N, M)
    for N, M in ((8, 1 << 18), (64, 65536), (512, 16384), (1024, 4096), (4096, 256), (1, 1 << 20)):
        assert direct(N, M, 1000), (N, M)
    for N, M in ((2, 1 << 20), (20, 1 << 18), (64, 1 << 18), (200, 65536), (100, 65536), (1024, 8192), (4096, 700)):
        took = [direct(N, M, ids) for ids in (0, 1, 12, 100, 300, 1000, 3000, 10000, 10**5, 10**6)]
        assert took == sorted(took, reverse=True), (N, M)  # longer rows never return to it
        assert not took[-1]
    assert not direct(257, 4096, 12, ta=16) and not direct(4097, 256, 12) and not direct(1025, 1 << 13, 12)


def test_regrouping_covers_batches_whose_rows_may_resemble_each_other(rules):
    """Regrouping is left out only where its kernels cost a tenth of the sweep or more, whatever the number of rows."""
    for N, M, ids in ((64000, 4096, 12), (16000, 16384, 12), (4000, 65536, 12), (8000, 65536, 12), (512000, 484, 12),
                      (30000, 4096, 200), (500000, 1 << 20, 12), (200, 1 << 20, 12)):
        assert rules.regroups(N, M, N * ids, 8), (N, M, ids)
    for N, M, ids in ((85000, 25, 100), (300000, 256, 100)):  # long rows gain on the smallest maps too
        assert rules.regroups(N, M, N * ids, 8), (N, M, ids)
    for N, M, ids in ((32000, 4096, 12), (2000, 65536, 12), (2000000, 256, 12), (128000, 484, 12), (10000, 256, 12),
                      (20000, 256, 100), (2000000, 256, 47)):
        assert not rules.regroups(N, M, N * ids, 8), (N, M, ids)


def test_no_search_without_a_plan_where_phases_regroup(rules):
    """A workspace that a search without a plan leaves holds the rows in the order given, as the phases must read it."""
    for ta in (8, 16, 32):
        for M in (1, 256, 257, 700, 4096, 32768, 32769, 65536, 131073, 1 << 18, 1 << 20):
            for N in (1, 2, 8, 48, 64, 256, 257, 1024, 1025, 4096, 4097, 10**6):
                for ids in (0, 1, 12, 100, 400, 1000, 4000, 15000, 30000):
                    if N * ids >= 2**31:
                        continue
                    if rules.regroups(N, M, N * ids, ta):
                        assert not any(rules.rows_direct(N, M, N * ids, ta, f16) for f16 in (0, 1)), (N, M, ids, ta)
