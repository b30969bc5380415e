"""The choice between windows in LDS and gathers through the L2 for long rows by column windows (the functions that the device
decides by, called on the host): which is taken where the two measured far apart, and what rules the windows in LDS out.
No GPU."""
import ctypes

import numpy as np
import pytest

from paper_2209_02882_amd import binding


def plan(op, K, N, rows, entries, longest, nnz=None, apart=0, worst=0, window_kb=0, max_long_rows=0, cus=256):
    """(in LDS, groups, shares per die, columns of a window, clocks in LDS, clocks of gathers)"""
    ints, clocks = [ctypes.c_int() for _ in range(4)], [ctypes.c_double() for _ in range(2)]
    status = binding.load().sgap_debug_plan_windows(int(op == "sddmm"), K, N, rows, entries, longest, nnz or entries, apart, worst,
                                                    window_kb, max_long_rows, cus, *map(ctypes.byref, ints + clocks))
    assert status == binding.SGAP_OK
    return [x.value for x in ints + clocks]


def skewed(op, rows, longest, N, **more):
    """One row in a hundred is long, from a tenth of the longest on."""
    lengths = np.linspace(longest / 10, longest, rows // 100).astype(np.int64)
    return plan(op, rows, N, lengths.size, int(lengths.sum()), longest, **more)


# (faster by a tenth and more on the chip)
@pytest.mark.parametrize("op,rows,longest,in_lds,gathered", [
    ("spmm", 500_000, 20_000, (64, 128, 160, 256, 384, 512, 1024), ()),
    ("spmm", 500_000, 10_000, (128, 160, 256, 384, 512, 1024), ()),
    ("spmm", 500_000, 5_000, (), (64, 160)),
    ("spmm", 250_000, 8_000, (64, 128, 160, 256, 384, 1024), ()),
    ("spmm", 120_000, 15_000, (64, 128, 160, 256, 384, 512, 1024), ()),
    ("spmm", 120_000, 2_400, (1024,), (64, 160, 208, 256)),
    ("spmm", 60_000, 7_500, (64, 128, 384, 512, 1024), ()),
    ("spmm", 30_000, 3_750, (64, 128, 384, 512, 1024), ()),
    ("sddmm", 500_000, 20_000, (64, 96, 128, 160, 256), ()),
    ("sddmm", 500_000, 5_000, (), (64, 96, 160, 256)),
    ("sddmm", 250_000, 8_000, (64, 96, 128, 160, 256), ()),
    ("sddmm", 120_000, 15_000, (64, 96, 128, 160, 256), ()),
    ("sddmm", 60_000, 7_500, (64, 96, 128, 160, 256), ()),
    ("sddmm", 30_000, 3_750, (64, 96, 128, 160, 256), ()),
])
def test_the_faster_form_is_taken(op, rows, longest, in_lds, gathered):
    assert [N for N in in_lds + gathered if skewed(op, rows, longest, N)[0]] == list(in_lds)


# the gathering kernels take every entry once per 256 columns
def test_gathers_cost_as_often_as_they_are_made():
    assert skewed("spmm", 500_000, 20_000, 1024)[5] > 3.9 * skewed("spmm", 500_000, 20_000, 256)[5]


# byte offsets of rows in a window and of entries have 32 and 31 bits
@pytest.mark.parametrize("op,window_kb", [("spmm", 154), ("sddmm", 149)])
def test_sizes_that_32_bits_hold(op, window_kb):
    assert plan(op, 1 << 24, 64, 300, 300_000, 1_000, window_kb=window_kb)[0]
    assert not plan(op, (1 << 24) + 1, 64, 300, 300_000, 1_000, window_kb=window_kb)[0]
    assert plan(op, 9_000, 64, 300, 300_000, 1_000, nnz=(1 << 29) - 1, window_kb=window_kb)[0]
    assert not plan(op, 9_000, 64, 300, 300_000, 1_000, nnz=1 << 29, window_kb=window_kb)[0]


@pytest.mark.parametrize("op,most_kb,most_columns", [("spmm", 154, 616), ("sddmm", 149, 596)])
def test_the_window_that_the_caller_names(op, most_kb, most_columns):
    for window_kb, columns in ((1, 4), (most_kb, most_columns), (most_kb + 1, 0), (3072, 0)):
        p = plan(op, 9_000, 64, 300, 900_000, 4_000, window_kb=window_kb)
        assert (p[0], p[3]) == (columns > 0, columns)
    assert plan(op, 9_000, 64, 255, 900_000, 4_000, window_kb=most_kb)[0] == 0
    assert plan(op, 9_000, 60, 300, 900_000, 4_000, window_kb=most_kb)[0] == 0


# 20 entries of the longest row, four of a row in the mean at least; what is reckoned with is what the kernels have
@pytest.mark.parametrize("op,most", [("spmm", 616), ("sddmm", 596)])
def test_the_window_by_the_rows(op, most):
    K, n = 120_000, 1_200
    for mean, longest, columns in ((1_000, 1_500, most), (8_000, 8_000, 300), (8_000, 16_000, 150), (8_000, 100_000, 60)):
        assert plan(op, K, 64, n, n * mean, longest)[3] in (0, columns)
    assert plan(op, K, 64, n, n * 8_000, 8_000)[3] == 300
    assert plan(op, K, 64, n, n * 8_000, 30_000)[4] > 1.3 * plan(op, K, 64, n, n * 8_000, 8_000)[4]


def test_what_windows_would_not_serve_is_gathered():
    entries = 55_000_000
    for op in ("spmm", "sddmm"):
        for N in (64, 256):
            assert plan(op, 500_000, N, 5_000, entries, 20_000, apart=entries // 10_000)[0]
            assert not plan(op, 500_000, N, 5_000, entries, 20_000, apart=entries // 100)[0]
            assert not plan(op, 500_000, N, 5_000, entries, 20_000, apart=20_000, worst=20_000)[0]


# every row needs the ends of its shares: of one share per die at least
def test_the_workspace_has_room_for_the_pointers():
    # windows of 154 KiB: 1,500 rows of B of 64 columns in 3 of them, four pointers for each row of the list
    room = {rows: plan("spmm", 1_500, 64, rows, rows * 100, 160, window_kb=154, max_long_rows=8192)[0] for rows in (3_640, 3_641)}
    assert room == {3_640: 1, 3_641: 0}


def test_bad_arguments():
    ints, clocks = [ctypes.c_int() for _ in range(4)], [ctypes.c_double() for _ in range(2)]
    out = [ctypes.byref(x) for x in ints + clocks]
    call = binding.load().sgap_debug_plan_windows
    assert call(0, 9_000, 62, 300, 900_000, 4_000, 900_000, 0, 0, 0, 0, 256, *out) == binding.SGAP_ERR_INVALID_ARG
    assert call(0, 9_000, 64, 300, 900_000, 4_000, 800_000, 0, 0, 0, 0, 256, *out) == binding.SGAP_ERR_INVALID_ARG
    assert call(0, 9_000, 64, 300, 900_000, 4_000, 900_000, 0, 0, 0, 0, 256, *out[:5], None) == binding.SGAP_ERR_INVALID_ARG
