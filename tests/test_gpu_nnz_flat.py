"""Nnz-balanced serial by teams of lanes that go each at its own pace: rows that cross teams' and tiles' ends, that span many
tiles, runs of rows without entries longer than a tile's window, and every number of lanes.  Exact on integer values."""
import numpy as np
import pytest
import torch

import oracle
from paper_2209_02882_amd import binding
from paper_2209_02882_amd import workloads as wl

pytestmark = pytest.mark.gpu


def lengths(kind, rng):
    if kind == "ragged":
        return rng.integers(0, 40, 3001)
    if kind == "single":  # a row for every entry of a tile
        return np.ones(5000, np.int64)
    if kind == "tiles":  # rows of a tile, one entry less and more, and of many
        return np.array([1024, 1023, 1025, 0, 512, 511, 1, 256, 255, 257, 7000, 3, 0, 2048, 1, 0, 4100, 0, 0, 9])
    n = np.zeros(9000, np.int64)  # runs without entries at both ends and longer than 1,024 rows
    n[[1500, 1501, 2900, 2901, 2903, 6000]] = [5, 700, 2, 1, 1300, 64]
    n[3000:4500:3] = 1
    return n


@pytest.mark.parametrize("N", [16, 17, 29, 32, 36, 61, 64, 65, 100, 125, 128])
@pytest.mark.parametrize("kind", ["ragged", "single", "tiles", "runs"])
def test_rows_across_teams_and_tiles(kind, N):
    rng = np.random.default_rng(N)
    rowptr, colidx = wl.csr_from_lengths(rng, lengths(kind, rng), 8000)
    M, K = rowptr.size - 1, 8000
    vals, B = wl.fill_values(rng, colidx.size, True), wl.fill_values(rng, K * N, True).reshape(K, N)
    ref, _ = oracle.spmm_csr(M, K, N, rowptr, colidx, vals, B, nthreads=8, bound=False)
    d = [torch.from_numpy(x).cuda() for x in (rowptr, colidx, vals, B)]
    C = torch.empty((M, N), device="cuda")
    for g in (1, 32):
        for hint in (-1, int(rowptr[-1]), 1_000_000, 10**8):  # every tile size, and grids of any number of workgroups
            C.fill_(float("nan"))
            binding.sgap_spmm_csr_ex(M, K, N, *d, C, g, binding.SGAP_REDUCE_SERIAL, binding.SGAP_SCHED_NNZ_BALANCED, nnz_hint=hint)
            assert np.array_equal(C.cpu().numpy().astype(np.float64), ref), (g, hint)
