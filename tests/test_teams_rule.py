"""Which calls teams of lanes that go each at its own pace take: the sizes on both sides of every line of the rules, and what a caller
names for itself.  Host logic, no GPU."""
import ctypes

import pytest

from paper_2209_02882_amd import binding

ROW, NNZ = "row_split", "nnz_balanced"


def spmm(M, K, N, nnz, g, strategy, schedule, **knobs):
    config = binding.make_config(g, strategy, schedule, **knobs)
    return binding.load().sgap_debug_spmm_teams(M, K, N, nnz, ctypes.byref(config), 256)


def mttkrp(I, J, nnz, g, strategy, schedule):
    return binding.load().sgap_debug_mttkrp_teams(I, J, g, binding.STRATEGIES[strategy], binding.SCHEDULES[schedule], nnz)


@pytest.mark.parametrize("N,g,nnz,M,K,takes", [
    (24, 8, 300_000, 25_000, 10_000, 1), (24, 8, 299_999, 30_000, 10_000, 0), (24, 8, 300_001, 25_000, 10_000, 0),  # 12 to a row
    (24, 8, 600_000, 30_000, 10_000, 1), (24, 8, 599_999, 30_000, 10_000, 0), (64, 4, 600_000, 30_000, 10_000, 1), (23, 8, 700_000, 30_000, 10_000, 1),
    (23, 8, 699_999, 30_000, 10_000, 0), (32, 4, 300_000, 30_000, 10_000, 0), (33, 4, 300_000, 30_000, 10_000, 1), (20, 8, 300_000, 30_000, 10_000, 1),
    (19, 8, 300_000, 30_000, 10_000, 0), (17, 4, 700_000, 30_000, 10_000, 1), (16, 8, 700_000, 30_000, 10_000, 0), (16, 16, 700_000, 30_000, 10_000, 1),
    (12, 16, 700_000, 30_000, 10_000, 1), (11, 16, 700_000, 30_000, 10_000, 0), (48, 8, 1_050_000, 30_000, 10_000, 1), (48, 8, 1_050_001, 30_000, 10_000, 0),
    (64, 8, 600_000, 40_000, 131_072, 1), (64, 8, 600_000, 40_000, 131_073, 0), (40, 8, 600_000, 40_000, 300_000, 1), (65, 8, 600_000, 40_000, 10_000, 0),
])
def test_row_split_parallel(N, g, nnz, M, K, takes):
    assert spmm(M, K, N, nnz, g, "parallel", ROW) == takes
    for knobs in ({"block_size": 256}, {"persistent": 1}, {"tile_cols": 32}, {"rows_per_group": 1}, {"reduce_size": g // 2}):
        assert spmm(M, K, N, nnz, g, "parallel", ROW, **knobs) == 0
    assert spmm(M, K, N, -1, g, "parallel", ROW) == 0


@pytest.mark.parametrize("N,g,nnz,M,K,takes", [
    (4, 4, 500_000, 50_000, 100_000, 1), (4, 4, 499_999, 50_000, 100_000, 0), (4, 1, 500_000, 50_000, 100_000, 0), (4, 2, 500_000, 50_000, 100_000, 1),
    (1, 1, 1_400_000, 200_000, 100_000, 1), (11, 1, 1_399_999, 200_000, 100_000, 0), (12, 1, 500_000, 50_000, 100_000, 1), (48, 1, 600_000, 50_000, 100_000, 1),
    (48, 1, 600_001, 50_000, 100_000, 0), (49, 1, 800_000, 100_000, 32_000, 1), (64, 1, 800_000, 100_000, 24_000, 1), (64, 1, 800_000, 100_000, 114_688, 1),
    (64, 1, 800_000, 100_000, 114_689, 0), (65, 1, 800_000, 100_000, 10_000, 0), (128, 1, 800_000, 100_000, 20_000, 1), (128, 1, 800_000, 100_000, 10_000, 0),
])
def test_row_split_serial(N, g, nnz, M, K, takes):
    # (what four neighbouring rows together come first for has longer rows)
    assert spmm(M, K, N, nnz, g, "serial", ROW) == takes
    for knobs in ({"block_size": 256}, {"persistent": 1}, {"tile_cols": 32}):
        assert spmm(M, K, N, nnz, g, "serial", ROW, **knobs) == 0
    assert spmm(M, K, N, -1, g, "serial", ROW) == 0


@pytest.mark.parametrize("N,g,nnz,M,takes", [
    (16, 16, 250_000, 20_000, 1), (16, 16, 249_999, 20_000, 0), (17, 16, 10_000, 1000, 1), (15, 16, 300_000, 20_000, 0), (128, 16, 300_000, 20_000, 1),
    (129, 16, 300_000, 20_000, 0), (64, 64, 400_000, 2000, 0), (64, 32, 400_000, 2000, 1), (65, 64, 400_000, 2000, 1), (64, 64, 399_999, 2000, 1),
    (64, 16, -1, 20_000, 1),
])
def test_nnz_balanced_serial(N, g, nnz, M, takes):
    assert spmm(M, 10_000, N, nnz, g, "serial", NNZ) == takes
    assert spmm(M, 10_000, N, nnz, g, "serial", NNZ, nnz_tile=512) == 0
    assert spmm(M, 10_000, N, nnz, g, "parallel", NNZ) == 0


@pytest.mark.parametrize("J,g,nnz,I,takes", [
    (80, 8, -1, 1000, 1), (79, 8, -1, 1000, 0), (48, 4, 1, 1000, 1), (48, 2, 12_000, 1000, 1), (48, 2, 11_999, 1000, 0), (32, 8, 12_000, 1000, 1),
    (32, 8, 11_999, 1000, 0), (32, 8, 150_000, 100_000, 1), (31, 8, 149_999, 1000, 0), (20, 8, 150_000, 100_000, 1), (19, 8, 299_999, 1000, 0),
    (12, 8, 300_000, 100_000, 1), (11, 8, 400_000, 5000, 1), (11, 8, 400_000, 5001, 0), (11, 8, 399_999, 4000, 0), (1, 1, 400_000, 40_000, 1),
])
def test_mttkrp_by_slices(J, g, nnz, I, takes):
    assert mttkrp(I, J, nnz, g, "parallel", ROW) == takes
    assert mttkrp(I, J, nnz, g, "serial", ROW) == 0 and mttkrp(I, J, nnz, g, "parallel", NNZ) == 0


@pytest.mark.parametrize("J,nnz,takes", [(9, 1, 1), (8, 500_000, 1), (8, 499_999, 0), (4, 700_000, 1), (4, 699_999, 0), (3, 666_666, 1), (1, 1_999_999, 0), (1, -1, 1)])
def test_mttkrp_by_tiles(J, nnz, takes):
    assert mttkrp(1000, J, nnz, 8, "serial", NNZ) == takes


def test_arguments_are_checked():
    lib, config = binding.load(), binding.make_config(8, "serial", ROW)
    assert lib.sgap_debug_spmm_teams(0, 1, 1, 1, ctypes.byref(config), 256) == -1
    assert lib.sgap_debug_spmm_teams(1, 1, 1, 1, None, 256) == -1
    assert lib.sgap_debug_mttkrp_teams(1, 1, 3, 0, 0, 1) == -1 and lib.sgap_debug_mttkrp_teams(0, 1, 8, 0, 0, 1) == -1
