"""Teams of lanes where long rows lie together, and blocks of as many rows or slices as there may be.

Row-split parallel: in a block of more than 3,072 entries rows of 96 and more are a finder's, and the others of a piece close up; rows
at both sides of these numbers, first, last and one behind the other, in blocks of every size that the rule makes, and pieces that end
inside a row behind such rows.  Exact on integer values."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2209_02882_amd import binding
from paper_2209_02882_amd import workloads as wl

pytestmark = pytest.mark.gpu


def spmm_is_exact(rowptr, colidx, K, n, g, strategy, schedule, hints, rng):
    M = rowptr.size - 1
    vals, B = wl.fill_values(rng, colidx.size, True), wl.fill_values(rng, K * n, True).reshape(K, n)
    ref, _ = oracle.spmm_csr(M, K, n, rowptr, colidx, vals, B, nthreads=8, bound=False)
    d = [torch.from_numpy(x).cuda() for x in (rowptr, colidx, vals, B)]
    C = torch.empty((M, n), device="cuda")
    config = binding.make_config(g, strategy, schedule)
    for hint in hints:
        print("  rows", M, n, g, hint, flush=True)
        assert binding.load().sgap_debug_spmm_teams(M, K, n, hint, ctypes.byref(config), 256) == 1
        C.fill_(float("nan"))
        binding.sgap_spmm_csr_cfg(M, K, n, *d, C, config, nnz_hint=hint)
        assert np.array_equal(C.cpu().numpy().astype(np.float64), ref), hint


def lengths(kind, M, rng):
    if kind == "down":  # in order of their lengths
        return np.sort(1 + rng.geometric(0.02, M) * (rng.random(M) < 0.2) + rng.integers(0, 4, M))[::-1]
    n = rng.integers(0, 9, M)
    if kind == "among short ones":  # in some stretches two rows of three are a finder's
        for at in range(0, M, 4000):
            n[at:at + 300:3] = rng.integers(90, 768, 100)
            n[at + 1:at + 300:3] = rng.choice([94, 95, 96, 97, 767, 768, 769, 2500], 100)
        return n
    # stretches of 3,072 entries and one less and more in whatever block they are, of rows that are just not long enough, and what
    # follows a piece's end
    n[:] = 0
    for at in range(0, M - 400, 1700):
        n[at:at + 32] = 96
        n[at] += at % 3 - 1
        n[at + 200:at + 300] = 95
        n[at + 220] = 700
        n[at + 299] = 4000
    n[[0, M - 1]] = [767, 96]
    return n


@pytest.mark.parametrize("kind", ["down", "among short ones", "at the limits"])
@pytest.mark.parametrize("n,g", [(13, 32), (24, 8), (32, 16), (37, 4), (48, 8), (64, 8)])
def test_long_rows_together(kind, n, g):
    rng = np.random.default_rng(n)
    M, K = 60_000, 5000
    rowptr, colidx = wl.csr_from_lengths(rng, lengths(kind, M, rng), K)
    hints = [1_000_000, 1_200_000] if n < 24 else [300_000, 600_000] if n > 48 else [300_000, 500_000, 1_200_000]
    spmm_is_exact(rowptr, colidx, K, n, g, "parallel", "row_split", hints, rng)


@pytest.mark.parametrize("n,g,strategy,schedule", [(3, 4, "serial", "row_split"), (40, 1, "serial", "row_split"), (24, 8, "parallel", "row_split"),
                                                   (20, 8, "serial", "nnz_balanced")])
def test_blocks_of_as_many_rows_as_there_may_be(n, g, strategy, schedule):
    """1,024 rows to a block, most of them without entries."""
    rng = np.random.default_rng(n)
    M, K = 1_500_000, 900
    lengths = np.zeros(M, np.int64)
    lengths[rng.integers(0, M, 60_000)] = rng.integers(1, 9, 60_000)
    lengths[[0, 1023, 1024, 2047, 5000, M - 1]] = [1, 3, 2, 700, 900, 5]
    lengths[300_000:300_700] = 4  # a piece's entries end in front of its rows
    rowptr, colidx = wl.csr_from_lengths(rng, lengths, K)
    spmm_is_exact(rowptr, colidx, K, n, g, strategy, schedule, [500_000], rng)


@pytest.mark.parametrize("slices", [255 * 1024, 256 * 1024 - 3, 256 * 1024 + 1, 300_000])
def test_mttkrp_blocks_of_as_many_slices_as_there_may_be(slices):
    """255 slices to a block, 256, and no more."""
    rng = np.random.default_rng(slices)
    K, L, J, hint = 300, 200, 24, 150_000
    fibers = np.zeros(slices, np.int64)
    fibers[rng.integers(0, slices, 40_000)] = rng.integers(1, 4, 40_000)
    fibers[[0, 254, 255, 256, 511, 512, slices - 1]] = [2, 1, 3, 1, 2, 290, 4]
    fptr, fidx = wl.csr_from_lengths(rng, fibers, K)
    eptr, eidx = wl.csr_from_lengths(rng, rng.integers(0, 4, fidx.size), L)
    vals, X1, X2 = wl.fill_values(rng, eidx.size, True), *(wl.fill_values(rng, n * J, True).reshape(n, J) for n in (K, L))
    ref, _ = oracle.mttkrp_csf(slices, K, L, J, fptr, fidx, eptr, eidx, vals, X1, X2, nthreads=8)
    d = [torch.from_numpy(x).cuda() for x in (fptr, fidx, eptr, eidx, vals, X1, X2)]
    assert binding.load().sgap_debug_mttkrp_teams(slices, J, 8, binding.SGAP_REDUCE_PARALLEL, binding.SGAP_SCHED_ROW_SPLIT, hint) == 1
    Y = torch.full((slices, J), float("nan"), device="cuda")
    binding.sgap_mttkrp_csf_ex(slices, K, L, J, *d, Y, 8, binding.SGAP_REDUCE_PARALLEL, binding.SGAP_SCHED_ROW_SPLIT, nnz_hint=hint)
    assert np.array_equal(Y.cpu().numpy().astype(np.float64), ref)
