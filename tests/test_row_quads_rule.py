"""Which calls of the row-split schedule's serial strategy go by four neighbouring rows together.  Host logic, no GPU."""
import ctypes

import pytest

from paper_2209_02882_amd import binding


def by_quads(M, N, nnz_hint, group=1, strategy="serial", schedule="row_split", compute_units=256, **knobs):
    cfg = binding.make_config(group, strategy, schedule, **knobs)
    return binding.load().sgap_debug_row_quads(M, N, nnz_hint, ctypes.byref(cfg), compute_units)


# 64 lanes hold 256 columns, and the kernel makes one pass over a tile
@pytest.mark.parametrize("N,tile_cols,want", [(256, 256, 1), (512, 256, 1), (512, 0, 1), (260, 260, 0), (300, 300, 0), (300, 1000, 0), (520, 512, 0),
                                              (520, 257, 0), (10_000, 128, 1), (128, 1000, 1)])
def test_a_tile_fits_one_pass(N, tile_cols, want):
    assert by_quads(1_000_000, N, 20_000_000, tile_cols=tile_cols) == want


@pytest.mark.parametrize("N,tile_cols,rows", [(33, 0, 64), (64, 0, 64), (65, 0, 32), (128, 0, 32), (129, 0, 32), (256, 256, 16), (128, 48, 64)])
def test_enough_blocks_of_rows(N, tile_cols, rows):
    for units in (1, 8, 256, 304):
        least = (8 if rows == 64 else 5) * units * rows
        for group in (1, 2, 4):
            assert by_quads(least, N, 20 * least, group, compute_units=units, tile_cols=tile_cols) == 1
            assert by_quads(least - 1, N, 20 * least, group, compute_units=units, tile_cols=tile_cols) == 0


def test_rows_of_such_a_length_in_the_mean():
    M = 1_000_000
    assert [by_quads(M, 128, n * M) for n in (1, 12, 13, 31, 32, 33)] == [0, 0, 1, 1, 1, 0]
    assert by_quads(M, 128, 12 * M + 1) == 1 and by_quads(M, 128, 32 * M + 1) == 0


def test_calls_that_name_their_own_way():
    M, nnz = 1_000_000, 20_000_000
    assert by_quads(M, 128, nnz) == 1 and by_quads(M, 128, nnz, reduce_size=1) == 1 and by_quads(M, 128, nnz, xcd_remap=0) == 1
    assert by_quads(M, 128, -1) == 0 and by_quads(M, 128, 0) == 0  # nobody knows how many entries there are
    assert by_quads(M, 128, nnz, group=8) == 0
    assert by_quads(M, 128, nnz, strategy="parallel") == 0 and by_quads(M, 128, nnz, schedule="nnz_balanced") == 0
    assert by_quads(M, 128, nnz, block_size=256) == 0 and by_quads(M, 128, nnz, persistent=1) == 0
    assert by_quads(M, 32, nnz) == 0 and by_quads(M, 128, nnz, tile_cols=32) == 0  # fewer than 16 lanes
    assert by_quads(M, 3, nnz) == 0
    assert by_quads(0, 128, nnz) == -1 and by_quads(M, 128, nnz, block_size=100) == -1
