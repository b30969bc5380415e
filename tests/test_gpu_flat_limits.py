"""Teams of lanes that go each at its own pace, in every kernel that has them: operands on both sides of 4 GiB, and values that
are not finite in the first row of a dense operand, which entries that are left out of a load must not bring in."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2209_02882_amd import binding
from paper_2209_02882_amd import workloads as wl

pytestmark = pytest.mark.gpu

ROWS, COLS = 50_000, 6200
LONG = [768, 700, 4096, 33, 1500, 2561]
SPMM = [  # the kernel, columns, (strategy, schedule, count of entries that the library is told)
    ("row-split serial, short rows", n, (binding.SGAP_REDUCE_SERIAL, binding.SGAP_SCHED_ROW_SPLIT, 500_000)) for n in (1, 3, 5, 24, 33)
] + [
    ("row-split parallel, shared blocks", n, (binding.SGAP_REDUCE_PARALLEL, binding.SGAP_SCHED_ROW_SPLIT, hint))
    for n, hint in ((13, 1_000_000), (24, 500_000), (37, 500_000), (40, 500_000))
] + [
    ("row-split parallel, rows that a workgroup takes with fewer loads in flight", n, (binding.SGAP_REDUCE_PARALLEL, binding.SGAP_SCHED_ROW_SPLIT, 1_800_000))
    for n in (24, 37)
] + [
    ("row-split parallel, rows that a workgroup takes", n, (binding.SGAP_REDUCE_PARALLEL, binding.SGAP_SCHED_ROW_SPLIT, 200_000))
    for n in (1, 3, 6, 37, 48, 100)
] + [
    ("nnz-balanced serial", n, (binding.SGAP_REDUCE_SERIAL, binding.SGAP_SCHED_NNZ_BALANCED, 700_000)) for n in (16, 37, 64, 125)
]


def matrix(n, seed):
    rng = np.random.default_rng(seed)
    lengths = rng.integers(0, 9, ROWS)
    lengths[rng.integers(0, ROWS, 60)] = np.resize(LONG, 60)
    rowptr, colidx = wl.csr_from_lengths(rng, lengths, COLS)
    return rowptr, colidx, wl.fill_values(rng, colidx.size, True), wl.fill_values(rng, COLS * n, True).reshape(COLS, n)


def spmm(point, rowptr, colidx, vals, B, n, g=16):
    strategy, schedule, hint = point
    C = torch.full((ROWS, n), float("nan"), device="cuda")
    rp, ci, va = (torch.from_numpy(x).cuda() for x in (rowptr, colidx, vals))
    binding.sgap_spmm_csr_ex(ROWS, B.shape[0], n, rp, ci, va, B, C, g, strategy, schedule, nnz_hint=hint)
    return C.cpu().numpy().astype(np.float64)


def far(x):
    """x with rows of zeros in front of it, so that its middle lies at 4 GiB, and how many."""
    first = 2**32 // (4 * x.shape[1]) - x.shape[0] // 2
    wide = torch.zeros((first + x.shape[0], x.shape[1]), device="cuda")
    wide[first:] = torch.from_numpy(x)
    return wide, np.int32(first)


@pytest.mark.parametrize("kernel,n,point", SPMM)
def test_spmm_teams_are_the_kernel(kernel, n, point):
    strategy, schedule, hint = point
    names = [{v: k for k, v in d.items()}[x] for d, x in ((binding.STRATEGIES, strategy), (binding.SCHEDULES, schedule))]
    config = binding.make_config(16, *names)
    for K in (COLS, 2**32 // (4 * n) + COLS // 2):
        assert binding.load().sgap_debug_spmm_teams(ROWS, K, n, hint, ctypes.byref(config), 256) == (0 if "workgroup" in kernel else 1)


@pytest.mark.parametrize("kernel,n,point", SPMM)
def test_spmm_offsets_of_64_bits(kernel, n, point):
    rowptr, colidx, vals, B = matrix(n, n)
    ref, _ = oracle.spmm_csr(ROWS, COLS, n, rowptr, colidx, vals, B, nthreads=8, bound=False)
    wide, first = far(B)
    assert np.array_equal(spmm(point, rowptr, colidx + first, vals, wide, n), ref)


@pytest.mark.parametrize("kernel,n,point", SPMM)
def test_spmm_first_row_not_finite(kernel, n, point):
    rowptr, colidx, vals, B = matrix(n, n)
    vals[vals == 0] = 1
    B[0], B[4000] = np.nan, np.inf
    got = spmm(point, rowptr, colidx, vals, torch.from_numpy(B).cuda(), n)
    names = lambda col: np.bincount(np.repeat(np.arange(ROWS), np.diff(rowptr))[colidx == col], minlength=ROWS) > 0
    with_0, with_4000 = names(0), names(4000)
    assert with_0.any() and (with_4000 & ~with_0).any()
    assert np.isnan(got[with_0]).all() and np.isinf(got[with_4000 & ~with_0]).all()
    B[0] = B[4000] = 0
    ref, _ = oracle.spmm_csr(ROWS, COLS, n, rowptr, colidx, vals, B, nthreads=8, bound=False)
    rest = ~with_0 & ~with_4000
    assert np.array_equal(got[rest], ref[rest])


MTTKRP = [("slices", j, (binding.SGAP_REDUCE_PARALLEL, binding.SGAP_SCHED_ROW_SPLIT, None)) for j in (1, 3, 6, 32, 37)] + [
    ("slices by teams", j, (binding.SGAP_REDUCE_PARALLEL, binding.SGAP_SCHED_ROW_SPLIT, 1_000_000)) for j in (1, 3, 6, 32, 37)] + [
    ("tiles", j, (binding.SGAP_REDUCE_SERIAL, binding.SGAP_SCHED_NNZ_BALANCED, -1)) for j in (1, 3, 6, 32, 37)] + [
    ("shares", j, (binding.SGAP_REDUCE_SERIAL, binding.SGAP_SCHED_NNZ_BALANCED, None)) for j in (1, 3, 6, 8)]
SLICES, EXTENT = 2500, 4000


def tensor(j, seed):
    rng = np.random.default_rng(seed)
    fibers = rng.integers(0, 5, SLICES)
    fibers[[7, 1000]] = [700, 90]
    fptr, fidx = wl.csr_from_lengths(rng, fibers, EXTENT)
    entries = rng.integers(1, 9, int(fptr[-1]))
    entries[rng.integers(0, entries.size, 30)] = np.resize([33, 100, 400, 3400], 30)
    eptr, eidx = wl.csr_from_lengths(rng, entries, EXTENT)
    X1, X2 = (wl.fill_values(rng, EXTENT * j, True).reshape(EXTENT, j) for _ in range(2))
    return fptr, fidx, eptr, eidx, wl.fill_values(rng, eidx.size, True), X1, X2


def mttkrp(point, t, X1, X2, j):
    strategy, schedule, hint = point
    fptr, fidx, eptr, eidx, vals = (torch.from_numpy(x).cuda() for x in t)
    Y = torch.full((SLICES, j), float("nan"), device="cuda")
    binding.sgap_mttkrp_csf_ex(SLICES, X1.shape[0], X2.shape[0], j, fptr, fidx, eptr, eidx, vals, X1, X2, Y, 8, strategy, schedule,
                               nnz_hint=eidx.numel() if hint is None else hint)
    return Y.cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("kernel,j,point", MTTKRP)
def test_mttkrp_offsets_of_64_bits(kernel, j, point):
    fptr, fidx, eptr, eidx, vals, X1, X2 = tensor(j, j)
    ref, _ = oracle.mttkrp_csf(SLICES, EXTENT, EXTENT, j, fptr, fidx, eptr, eidx, vals, X1, X2, nthreads=8)
    (wide1, first1), (wide2, first2) = far(X1), far(X2)
    got = mttkrp(point, (fptr, fidx + first1, eptr, eidx + first2, vals), wide1, wide2, j)
    assert np.array_equal(got, ref)


@pytest.mark.parametrize("kernel,j,point", MTTKRP)
def test_mttkrp_first_rows_not_finite(kernel, j, point):
    fptr, fidx, eptr, eidx, vals, X1, X2 = tensor(j, j)
    X1[0], X2[0] = np.nan, np.inf
    got = mttkrp(point, (fptr, fidx, eptr, eidx, vals), torch.from_numpy(X1).cuda(), torch.from_numpy(X2).cuda(), j)
    fiber_of = np.repeat(np.arange(fidx.size), np.diff(eptr))
    bad_fiber = (fidx == 0) | (np.bincount(fiber_of[eidx == 0], minlength=fidx.size) > 0)
    bad = np.bincount(np.repeat(np.arange(SLICES), np.diff(fptr))[bad_fiber], minlength=SLICES) > 0
    assert bad.any() and not bad.all()
    X1[0] = X2[0] = 0
    ref, _ = oracle.mttkrp_csf(SLICES, EXTENT, EXTENT, j, fptr, fidx, eptr, eidx, vals, X1, X2, nthreads=8)
    assert np.array_equal(got[~bad], ref[~bad])
    assert not np.isfinite(got[np.bincount(np.repeat(np.arange(SLICES), np.diff(fptr))[fidx == 0], minlength=SLICES) > 0]).any()
