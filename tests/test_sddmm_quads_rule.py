"""Which matrices the parallel strategy of SDDMM takes by four neighbouring rows together.  Host logic, no GPU."""
import numpy as np
import pytest

from paper_2209_02882_amd import binding


def by_quads(rowptr, colidx, J, g, K=None, hint=None):
    return binding.load().sgap_debug_sddmm_quads(rowptr.size - 1, K or int(colidx.max()) + 1, J, g, colidx.size if hint is None else hint,
                                                 rowptr.ctypes.data, colidx.ctypes.data)


def from_lengths(lengths, columns=None):
    """Rows of that many neighbouring columns, or of columns without order."""
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    row = np.repeat(np.arange(lengths.size), lengths)
    if columns is None:
        return rowptr, (row + np.arange(row.size) - rowptr[row]).astype(np.int32)
    return rowptr, np.sort(columns(row.size)).astype(np.int32)


def bands(one_in, long=40, rows=200_000, clustered=1):
    lengths = np.full(rows, 27)
    if one_in:
        chosen = np.random.default_rng(one_in).random(rows // clustered) < 1 / one_in
        lengths[:chosen.size * clustered][np.repeat(chosen, clustered)] = long
    return from_lengths(lengths)


@pytest.mark.parametrize("J,g", [(72, 8), (100, 16), (128, 8), (128, 16), (128, 32), (200, 16), (256, 64)])
def test_rows_alike_go_by_four(J, g):
    assert by_quads(*bands(0), J, g) == 1
    assert by_quads(*bands(200), J, g) == 1


# a row of 32 entries or more leaves its whole quad to a way that costs more than the others gain
@pytest.mark.parametrize("J,g", [(72, 8), (100, 16), (128, 8), (128, 16), (128, 32), (200, 16), (256, 64)])
@pytest.mark.parametrize("one_in,clustered", [(8, 1), (8, 3), (4, 3), (3, 1)])
def test_rows_of_a_mesh_of_which_many_are_long_go_entry_by_entry(one_in, clustered, J, g):
    assert by_quads(*bands(one_in, clustered=clustered), J, g) == 0
    assert by_quads(*bands(one_in, long=32, clustered=clustered), J, g) == 0


def test_wide_rows_bear_a_few_more_long_ones():
    rowptr, colidx = bands(29)
    assert by_quads(rowptr, colidx, 100, 8) == 0 and by_quads(rowptr, colidx, 200, 16) == 1


@pytest.mark.parametrize("J,g", [(100, 8), (256, 16)])
def test_columns_without_order_go_entry_by_entry(J, g):
    rng = np.random.default_rng(1)
    lengths = np.full(120_000, 20)
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    colidx = np.sort(rng.integers(0, 120_000, (lengths.size, 20)), axis=1).ravel().astype(np.int32)
    assert by_quads(rowptr, colidx, J, g) == 0


@pytest.mark.parametrize("shared,J,g,want", [(10, 100, 8, 0), (12, 100, 8, 1), (9, 200, 16, 0), (10, 200, 16, 1)])
def test_how_much_neighbours_share(shared, J, g, want):
    rows = 120_000
    columns = np.concatenate([np.tile(np.arange(shared), (rows, 1)), 100 + 20 * (np.arange(rows)[:, None] % 50) + np.arange(20 - shared)], axis=1)
    rowptr = (20 * np.arange(rows + 1)).astype(np.int32)
    assert by_quads(rowptr, columns.ravel().astype(np.int32), J, g) == want


def test_calls_that_do_not_look():
    rowptr, colidx = bands(0)
    assert by_quads(rowptr, colidx, 100, 8, hint=-1) == 0  # nobody knows how many entries there are
    assert by_quads(rowptr, colidx, 100, 8, hint=1_499_999) == 0
    for g, least in ((8, 68), (16, 68), (32, 72), (16, 132), (32, 132), (64, 136)):  # narrow
        assert by_quads(rowptr, colidx, least - 1, g) == 0 and by_quads(rowptr, colidx, least, g) == 1
    assert by_quads(rowptr, colidx, 100, 4) == 0 and by_quads(rowptr, colidx, 100, 64) == 0  # lanes and steps of an entry
    assert by_quads(rowptr, colidx, 128, 8, K=2**23) == 0 and by_quads(rowptr, colidx, 128, 8, K=2**23 - 1) == 1  # offsets of 32 bits
    assert by_quads(rowptr, colidx, 0, 8) == 0
    assert by_quads(rowptr, colidx, 100, 3) == -1 and by_quads(rowptr, colidx, -1, 8) == -1
