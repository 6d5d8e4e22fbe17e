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


I = ctypes.c_int
lane_mfma_offs_at = _planner("_ZN5lloyd17lane_mfma_offs_atEiii", ctypes.c_size_t, I, I, I)


@pytest.mark.parametrize("W", [1, 2, 4, 8])
def test_offset_table_of_the_lane_kernel_is_aligned(W):
    """It is read 16 bytes at a time; the counts before it are W (K + 1) ints."""
    off = [(M, K) for K in range(1, 65) for M in range(1, 33) if lane_mfma_offs_at(M, K, W) % 16]
    assert off == []
