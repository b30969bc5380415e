"""Column counts that the columns per lane do not divide, and rows that a whole workgroup of the
row-split schedule takes together: exact on integer-valued inputs."""
import numpy as np
import pytest
import torch

import oracle
from paper_2209_02882_amd import binding
from paper_2209_02882_amd import workloads as wl

from gpu_util import DeviceProblem

pytestmark = pytest.mark.gpu


def problem(M, K, N, lengths, seed):
    rng = np.random.default_rng(seed)
    rowptr, colidx = wl.csr_from_lengths(rng, np.asarray(lengths), K)
    return wl.SpmmProblem("ragged", M, K, N, rowptr, colidx, wl.fill_values(rng, colidx.size, True),
                          wl.fill_values(rng, K * N, True).reshape(K, N)), rng


# a group of G lanes shares rows from max(256, 96 * G / passes over the columns) entries on
@pytest.mark.parametrize("N", [1, 3, 4, 5, 37, 64, 131, 300])
def test_rows_that_a_workgroup_shares(N):
    lengths = [0, 255, 256, 257, 3, 2047, 2048, 2049, 0, 1, 4096, 4500, 767, 768, 1535, 1536, 12] + [2] * 60 + [6143, 6144]
    p, _ = problem(len(lengths), 7000, N, lengths, seed=N)
    ref, _ = oracle.spmm_csr(p.M, p.K, p.N, p.rowptr, p.colidx, p.vals, p.B, nthreads=8, bound=False)
    dp = DeviceProblem(p)
    for g in binding.GROUP_SIZES:
        for knobs in ({}, {"block_size": 128}, {"block_size": 512, "rows_per_group": 5}, {"tile_cols": 8}, {"persistent": 1}):
            got = dp.run_cfg(binding.make_config(g, "parallel", "row_split", **knobs)).cpu().numpy()
            assert np.array_equal(got.astype(np.float64), ref), (g, knobs)


@pytest.mark.parametrize("J", [1, 2, 3, 5, 7, 33, 66, 127])
def test_ragged_columns_of_sddmm(J):
    p, rng = problem(200, 300, J, np.random.default_rng(J).integers(0, 60, 200), seed=J)
    X1 = wl.fill_values(rng, p.M * J, True).reshape(p.M, J)
    ref, _ = oracle.sddmm_csr(p.M, p.K, J, p.rowptr, p.colidx, p.vals, X1, p.B, nthreads=8, bound=False)
    dp = DeviceProblem(p)
    X1d = torch.from_numpy(X1).cuda()
    for st in ("parallel", "serial"):
        for g in binding.GROUP_SIZES:
            assert np.array_equal(dp.run_sddmm(X1d, g, st).cpu().numpy().astype(np.float64), ref), (g, st)


# long rows looked for over several rounds of a workgroup, next to each other and at both ends
@pytest.mark.parametrize("M,block", [(64, 128), (65, 256), (16385, 256), (400_000, 128), (400_000, 512)])
def test_long_rows_found_in_large_matrices(M, block):
    lengths = np.random.default_rng(M).integers(0, 3, M)
    where = np.array([0, 1, 2, 63, 64, M // 2, M // 2 + 1, M - 200, M - 1]) % M
    lengths[where] = [900, 256, 768, 1536, 255, 2500, 300, 1000, 767]
    p, _ = problem(M, 3000, 5, lengths, seed=M)
    ref, _ = oracle.spmm_csr(p.M, p.K, p.N, p.rowptr, p.colidx, p.vals, p.B, nthreads=8, bound=False)
    dp = DeviceProblem(p)
    for g in (2, 8, 32):
        got = dp.run_cfg(binding.make_config(g, "parallel", "row_split", block_size=block)).cpu().numpy()
        assert np.array_equal(got.astype(np.float64), ref), g


# chunk lanes that divide neither a wavefront nor a workgroup (2, 3, 5, 13, 25 and 63 of them; 64 and a second pass)
@pytest.mark.parametrize("N", [6, 9, 20, 52, 100, 252, 260])
def test_shared_rows_on_any_number_of_lanes(N):
    p, _ = problem(40, 7000, N, [256, 2049, 300, 4100, 0, 5] * 6 + [2047, 2048, 1, 383], seed=N)
    ref, _ = oracle.spmm_csr(p.M, p.K, p.N, p.rowptr, p.colidx, p.vals, p.B, nthreads=8, bound=False)
    dp = DeviceProblem(p)
    for g in (2, 16):
        for block in (0, 128, 512):
            got = dp.run_cfg(binding.make_config(g, "parallel", "row_split", block_size=block)).cpu().numpy()
            assert np.array_equal(got.astype(np.float64), ref), (g, block)
