"""The grid of a row-split launch: who looks for the rows that whole workgroups take, and who walks the others.  Host
logic, no GPU."""
import ctypes

import pytest

from paper_2209_02882_amd import binding

NEVER = 2**31 - 1


def plan(g, passes, M, items, nnz_hint, resident=0, dies=8, cus=256):
    out = [ctypes.c_int64() for _ in range(4)]
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
                    share_from, finders, walk_from, grid = plan(g, passes, M, items, hint, resident, dies)
                    assert (finders == 0) == (share_from == NEVER)
                    if g == 1 or 0 <= hint < max(256, 96 * g // passes):
                        assert finders == 0
                    else:
                        assert share_from == max(256, 96 * g // passes) and finders > 0
                    # every die has workgroups that walk, and the same number of them
                    assert 0 <= walk_from < grid and (grid - walk_from) % dies == 0 and walk_from % dies == 0
                    if resident:
                        # nothing on top of what the chip holds at once (a round of the dies at least)
                        assert walk_from == 0 and finders <= grid <= max(resident, dies)
                    else:
                        assert walk_from == finders and grid - walk_from >= items


def test_bad_arguments():
    lib = binding.load()
    x = ctypes.byref(ctypes.c_int64())
    assert lib.sgap_debug_plan_row_split(3, 1, 1, 1, 8, 256, -1, 0, x, x, x, x) == binding.SGAP_ERR_INVALID_ARG
    assert lib.sgap_debug_plan_row_split(8, 1, 1, 1, 8, 256, -2, 0, x, x, x, x) == binding.SGAP_ERR_INVALID_ARG
    assert lib.sgap_debug_plan_row_split(8, 1, 1, 1, 8, 256, -1, 0, x, x, x, None) == binding.SGAP_ERR_INVALID_ARG
