"""Row-split serial on short rows by teams of lanes that go each at its own pace: pieces of a block (2,560 entries, 1,024
rows), rows that a piece has no room for, rows without entries, and column tiles.  Exact on integer values."""
import numpy as np
import pytest
import torch

import oracle
from paper_2209_02882_amd import binding
from paper_2209_02882_amd import workloads as wl

pytestmark = pytest.mark.gpu

HINT = 500_000  # from so many entries on


def lengths(kind, M, rng):
    if kind == "ragged":
        return rng.integers(0, 17, M)
    if kind == "sparse":  # more rows than a piece holds before the entries fill it
        n = np.zeros(M, np.int64)
        n[rng.integers(0, M, M // 20)] = 1
        return n
    n = rng.integers(0, 9, M)  # and long rows at a piece's edges
    n[[0, 1, 5, 700, 701, 9_000, M // 2, M - 2, M - 1]] = [2559, 2560, 2561, 5121, 0, 2556, 7000, 1, 2560]
    return n


# (lanes of a team that divide nothing, one to three columns, a second pass over the columns is never taken by this kernel)
@pytest.mark.parametrize("kind,M,K,N", [("ragged", 65_001, 9_000, 24), ("ragged", 70_000, 3_000, 1), ("ragged", 65_000, 40_000, 64),
                                        ("sparse", 80_000, 500, 2), ("long", 60_001, 8_000, 33), ("long", 60_000, 8_000, 3),
                                        ("long", 50_000, 20_000, 96), ("long", 50_000, 8_000, 7), ("long", 50_000, 9_000, 64)])
def test_rows_by_teams(kind, M, K, N):
    rng = np.random.default_rng(M + N)
    rowptr, colidx = wl.csr_from_lengths(rng, lengths(kind, M, rng), K)
    vals, B = wl.fill_values(rng, colidx.size, True), wl.fill_values(rng, K * N, True).reshape(K, N)
    ref, _ = oracle.spmm_csr(M, K, N, rowptr, colidx, vals, B, nthreads=8, bound=False)
    d = [torch.from_numpy(x).cuda() for x in (rowptr, colidx, vals, B)]
    C = torch.empty((M, N), device="cuda")
    for g in (1, 2, 64):
        for hint in (HINT, max(HINT, int(rowptr[-1])), 12 * M):
            C.fill_(float("nan"))
            binding.sgap_spmm_csr_ex(M, K, N, *d, C, g, binding.SGAP_REDUCE_SERIAL, binding.SGAP_SCHED_ROW_SPLIT, nnz_hint=hint)
            assert np.array_equal(C.cpu().numpy().astype(np.float64), ref), (g, hint)
