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
