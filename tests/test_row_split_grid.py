"""The grid of a row-split launch: who looks for the rows that whole workgroups take, and who walks the others.  Host
logic, no GPU."""
import ctypes

import numpy as np
import pytest

from paper_2209_02882_amd import binding

NEVER = 2**31 - 1


def plan(g, passes, M, items, nnz_hint, resident=0, dies=8, cus=256):
    out = [ctypes.c_int64() for _ in range(5)]
    assert binding.load().sgap_debug_plan_row_split(g, passes, M, items, dies, cus, nnz_hint, resident,
                                                    *(ctypes.byref(x) for x in out)) == 0
    return tuple(x.value for x in out)


@pytest.mark.parametrize("dies", [8, 1])
@pytest.mark.parametrize("M,items", [(1, 1), (64, 3), (65, 100), (1000, 250), (1_000_000, 60_000), (2**31 - 2, 2**28)])
def test_rows_are_left_out_only_where_somebody_looks_for_them(M, items, dies):
    for g in binding.GROUP_SIZES:
        for passes in (1, 2, 75):
            for hint in (-1, 0, 1, 100, 255, 256, 5000, 2**31 - 65536):
                for resident in (0, 1, 7, 8, 1000, 2048):
                    share_from, finders, team, walk_from, grid = plan(g, passes, M, items, hint, resident, dies)
                    assert (finders == 0) == (share_from == NEVER)
                    if g == 1 or 0 <= hint < max(256, 96 * g // passes):
                        assert finders == 0
                    else:
                        assert share_from == max(256, 96 * g // passes) and finders > 0
                    assert team in (1, 2) and finders % team == 0
                    if team > 1:
                        assert 2 * -(-M // finders) <= 256 and finders <= 4 * 256 + dies
                    # every die has workgroups that walk, and the same number of them
                    assert 0 <= walk_from < grid and (grid - walk_from) % dies == 0 and walk_from % dies == 0
                    if resident:
                        # nothing on top of what the chip holds at once (a round of the dies at least)
                        assert walk_from == 0 and finders <= grid <= max(resident, dies)
                    else:
                        assert walk_from == finders and grid - walk_from >= items


def finder_rows(M, finders, i):
    lib = binding.load()
    n = lib.sgap_debug_finder_rows(M, finders, i, None, 0)
    rows = np.empty(max(n, 1), np.int64)
    assert lib.sgap_debug_finder_rows(M, finders, i, rows.ctypes.data, n) == n
    return rows[:n]


@pytest.mark.parametrize("M,finders", [(1, 1), (1, 8), (3, 8), (64, 8), (65, 8), (1000, 16), (50_021, 784), (65_536, 1024),
                                       (1_000_000, 2048), (2_097_152, 2048), (300_001, 7)])
def test_every_row_is_looked_at_by_one_finder_and_long_rows_fall_apart(M, finders):
    owner = np.full(M, -1)
    for i in range(finders):
        rows = finder_rows(M, finders, i)
        assert (owner[rows] == -1).all() and np.unique(rows).size == rows.size
        owner[rows] = i
    assert (owner >= 0).all()
    if finders < 64:
        return
    # neighbouring rows in bulk, and the longest rows of an R-MAT matrix: those with few one bits in their number
    for long_rows in (np.arange(finders), np.arange(M - finders, M)):
        assert np.bincount(owner[long_rows]).max() <= 16  # four units of four rows (equal stretches: 64 and more)
    bits = np.zeros(M, np.int64)
    for b in range(M.bit_length()):
        bits += np.arange(M) >> b & 1
    for few in (1, 2, 3):
        long_rows = np.flatnonzero(bits <= few)
        assert np.bincount(owner[long_rows]).max() <= 16 + 4 * long_rows.size / finders


def test_bad_arguments():
    lib = binding.load()
    assert lib.sgap_debug_finder_rows(0, 1, 0, None, 0) == -1
    assert lib.sgap_debug_finder_rows(10, 4, 4, None, 0) == -1
    assert lib.sgap_debug_finder_rows(10, 4, 0, None, 5) == -1
    x = ctypes.byref(ctypes.c_int64())
    assert lib.sgap_debug_plan_row_split(3, 1, 1, 1, 8, 256, -1, 0, x, x, x, x, x) == binding.SGAP_ERR_INVALID_ARG
    assert lib.sgap_debug_plan_row_split(8, 1, 1, 1, 8, 256, -2, 0, x, x, x, x, x) == binding.SGAP_ERR_INVALID_ARG
    assert lib.sgap_debug_plan_row_split(8, 1, 1, 1, 8, 256, -1, 0, x, x, x, x, None) == binding.SGAP_ERR_INVALID_ARG


@pytest.mark.parametrize("M,mean,most_rows", [(100_000, 16, 64), (2000, 100, 64), (2000, 200, 12), (2000, 400, 6), (2000, 5000, 4)])
def test_finders_look_at_fewer_rows_where_rows_are_long(M, mean, most_rows):
    _, finders, _, _, _ = plan(4, 1, M, M, M * mean)
    assert -(-M // finders) <= most_rows
