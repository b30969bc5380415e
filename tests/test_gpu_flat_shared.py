"""Row-split parallel by teams of lanes that share a block of rows: rows that several teams share and that go on in the next
piece (2,048 entries), those that are left to the workgroups in front of the grid (768 and more) first, last, alone and one
behind the other in a block, and blocks of rows without entries.  Exact on integer values."""
import numpy as np
import pytest
import torch

import oracle
from paper_2209_02882_amd import binding
from paper_2209_02882_amd import workloads as wl

pytestmark = pytest.mark.gpu

HINT = 700_000  # from so many entries on, whatever the columns


def lengths(kind, rng):
    if kind == "ragged":
        return rng.integers(0, 80, 20_001)
    if kind == "crowded":  # pieces that end inside rows, again and again
        n = np.zeros(8000, np.int64)
        n[::6] = rng.integers(500, 768, 1334)
        n[6 * rng.integers(0, 1334, 40)] = [768, 767, 769, 1300, 2048] * 8
        return n
    if kind == "sparse":  # blocks of as many rows as there may be
        n = np.zeros(1_400_000, np.int64)
        n[rng.integers(0, n.size, 3000)] = rng.integers(1, 900, 3000)
        return n
    n = rng.integers(0, 9, 30_000)
    n[[0, 1, 2, 40, 44, 45, 46, 90, 91, 5_000, 5_001, 5_003, 29_998, 29_999]] = [768, 767, 769, 4096, 33, 32, 2047, 2048, 2049, 700, 760, 765, 900, 768]
    n[10_000:10_200] = 768  # blocks of nothing else
    n[15_000:15_300:2] = 700
    return n


@pytest.mark.parametrize("kind,N", [("ragged", 12), ("ragged", 37), ("ragged", 64), ("crowded", 13), ("crowded", 32), ("crowded", 61), ("sparse", 12),
                                    ("long", 12), ("long", 24), ("long", 33), ("long", 64)])
def test_shared_blocks_of_rows(kind, N):
    rng = np.random.default_rng(N)
    K = 6000
    rowptr, colidx = wl.csr_from_lengths(rng, lengths(kind, rng), K)
    M = rowptr.size - 1
    vals, B = wl.fill_values(rng, colidx.size, True), wl.fill_values(rng, K * N, True).reshape(K, N)
    ref, _ = oracle.spmm_csr(M, K, N, rowptr, colidx, vals, B, nthreads=8, bound=False)
    d = [torch.from_numpy(x).cuda() for x in (rowptr, colidx, vals, B)]
    C = torch.empty((M, N), device="cuda")
    for g in (2, 32):
        for hint in (HINT, max(HINT, int(rowptr[-1])), 128 * M):  # down to blocks of few rows
            print("  rows", kind, N, g, hint, flush=True)
            C.fill_(float("nan"))
            binding.sgap_spmm_csr_ex(M, K, N, *d, C, g, binding.SGAP_REDUCE_PARALLEL, binding.SGAP_SCHED_ROW_SPLIT, nnz_hint=hint)
            assert np.array_equal(C.cpu().numpy().astype(np.float64), ref), (g, hint)
