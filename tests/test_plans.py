"""Launch plans and LDS layouts, asked of the library's planners on the host (no
GPU: a planner is arithmetic on n, M, K)."""
import ctypes

import pytest

import paper_1402_3788_amd as km


def _planner(name, restype, *argtypes):
    fn = getattr(km._lib, name)
    fn.restype = restype
    fn.argtypes = list(argtypes)
    return fn


class AccumPlan(ctypes.Structure):
    _fields_ = [("path", ctypes.c_int), ("waves", ctypes.c_int), ("groups", ctypes.c_int),
                ("accum", ctypes.c_int), ("list_cap", ctypes.c_int),
                ("lds_bytes", ctypes.c_size_t)]


I, I64 = ctypes.c_int, ctypes.c_int64
ASSIGN, ASSIGN_ACCUM, ACCUM_LABELS = 0, 1, 2
MAX_LDS = 160 * 1024
plan_lane_mfma = _planner("_ZN5lloyd14plan_lane_mfmaEliiNS_4ModeE", AccumPlan, I64, I, I, I)
plan_lane = _planner("_ZN5lloyd9plan_laneEliiNS_4ModeE", AccumPlan, I64, I, I, I)
plan_lane_l1 = _planner("_ZN5lloyd12plan_lane_l1Elii", AccumPlan, I64, I, I)
plan_tile = _planner("_ZN5lloyd9plan_tileEliiNS_4ModeE", AccumPlan, I64, I, I, I)
lane_mfma_offs_at = _planner("_ZN5lloyd17lane_mfma_offs_atEiii", ctypes.c_size_t, I, I, I)


@pytest.mark.parametrize("W", [1, 2, 4, 8])
def test_offset_table_of_the_lane_kernel_is_aligned(W):
    """It is read 16 bytes at a time; the counts before it are W (K + 1) ints."""
    off = [(M, K) for K in range(1, 65) for M in range(1, 33) if lane_mfma_offs_at(M, K, W) % 16]
    assert off == []


@pytest.mark.parametrize("mode", [ASSIGN, ASSIGN_ACCUM])
def test_lists_of_close_calls_fit(mode):
    """The capacity handed to the kernel is the one its LDS was sized for: the
    launch uses what the lists leave, and a list of the lane kernel holds the
    128 objects that it gathers there after an overflow."""
    for M, K in [(1, 5), (2, 64), (10, 8), (25, 16), (25, 64), (31, 33), (32, 64)]:
        for n in (1, 5_000, 40_000, 2_000_000):
            p = plan_lane_mfma(n, M, K, mode)
            assert 128 <= p.list_cap <= 2048 and p.lds_bytes <= MAX_LDS, (n, M, K)
            assert lane_mfma_offs_at(M, K, p.waves) % 16 == 0
            assert p.lds_bytes > p.waves * p.list_cap * 4
    for M, K in [(7, 40), (37, 100), (25, 256), (64, 186), (17, 545)]:
        for n in (1, 5_000, 2_000_000):
            p = plan_tile(n, M, K, mode)
            assert p.waves >= 1 and p.lds_bytes <= MAX_LDS, (n, M, K)
            assert p.lds_bytes > p.waves * p.list_cap * 8 >= 0


@pytest.mark.parametrize("M,K", [(25, 16), (10, 8), (3, 5), (64, 4), (25, 32)])
def test_l1_runs_of_few_objects_assign_and_sum_in_one_launch(M, K):
    """A plan spread over the compute units has few waves per workgroup because
    there are few tiles, not because LDS holds no more."""
    for n in (1, 5_000, 16_400, 20_000, 60_000, 98_304, 100_000, 150_000, 190_000):
        p = plan_lane_l1(n, M, K)
        assert p.waves >= 1, n
        assert p.waves * p.groups >= min((n + 63) // 64, p.waves * 256)


@pytest.mark.parametrize("M,K", [(4, 4), (10, 3), (25, 4), (25, 16), (64, 4)])
def test_few_tiles_are_spread_in_one_round(M, K):
    """Smaller workgroups only as long as no wave gets a second tile for it."""
    full = plan_lane(10**7, M, K, ASSIGN_ACCUM).waves
    for n in (64, 5_000, 20_000, 65_536, 65_600, 98_304, 98_368, 150_000, 300_000):
        p = plan_lane(n, M, K, ASSIGN_ACCUM)
        assert p.waves == full or p.waves * p.groups >= (n + 63) // 64, n
        assert p.groups <= 256


@pytest.mark.parametrize("mode,limit", [(ASSIGN, 768), (ASSIGN_ACCUM, 256), (ACCUM_LABELS, 256)])
@pytest.mark.parametrize("M,K", [(10, 8), (25, 16), (25, 32), (32, 64)])
def test_few_tiles_of_the_lane_kernel_are_spread_in_one_round(M, K, mode, limit):
    full = plan_lane_mfma(10**7, M, K, mode)
    assert full.groups <= limit
    for n in (64, 5_000, 16_384, 40_000, 65_536, 70_000, 100_000, 131_072, 131_136, 500_000):
        p = plan_lane_mfma(n, M, K, mode)
        assert p.waves == full.waves or p.waves * p.groups >= (n + 63) // 64, n
        assert p.groups <= full.groups, n


def test_sums_in_slices_fill_the_chip_within_lds():
    """Slices of 16, 8 or 4 features with the slabs of at least six waves, but
    where four features are all that fits."""
    plan_accum = _planner("_ZN5lloyd10plan_accumElii", AccumPlan, I64, I, I)
    for M, K in [(16, 1024), (15, 1000), (25, 400), (25, 655), (37, 200), (57, 140), (64, 20), (64, 256)]:
        for n in (1, 65, 16_384, 400_000, 10**7):
            p = plan_accum(n, M, K)
            assert p.accum in (4, 8, 16) and p.lds_bytes <= MAX_LDS and 1 <= p.groups <= 256
            slices = -(-M // p.accum)
            assert (p.groups - 1) * slices < 256
            if p.accum > 4:
                assert p.waves >= 6 and p.accum // 2 < M
                assert slices * -(-n // (64 * p.waves)) >= 256
    assert plan_accum(400_000, 57, 140).accum == 16
    assert plan_accum(16_384, 25, 400).accum == 4


@pytest.mark.parametrize("n,M,K", [(70_000, 17, 473), (16_384, 17, 525), (100_000, 18, 447),
                                   (100_000, 28, 295), (70_000, 22, 386), (20_011, 18, 525)])
def test_lists_do_not_push_few_objects_out_of_the_static_workspace(n, M, K):
    """Shapes whose partials fit it with the waves that LDS holds without lists."""
    for flags in (0, 4, 8):
        assert 0 < km.kmeans_workspace_bytes(n, M, K, flags) <= km.NOALLOC_MAX_WORKSPACE
