"""SDDMM on long rows whose windows of X2T lie in LDS (lists of at least 256 long rows, 64 <= J <= 256): exact on
integer-valued inputs, at the edges of teams, slots, column tiles, windows and shares.  A window_kb of at most 149 asks for
these windows at any size."""
import numpy as np
import pytest
import torch

import oracle
from paper_2209_02882_amd import binding
from paper_2209_02882_amd import workloads as wl

from gpu_util import TOL, DeviceProblem
from test_gpu_panels_lds import LDS_RUNS, crowded, problem, without_order

pytestmark = pytest.mark.gpu


def check(p, min_len, what, exact=True, window_kb=149, runs=1):
    X1 = wl.fill_values(np.random.default_rng(p.M), p.M * p.N, exact).reshape(p.M, p.N)
    ref, bnd = oracle.sddmm_csr(p.M, p.K, p.N, p.rowptr, p.colidx, p.vals, X1, p.B, nthreads=8)
    dp = DeviceProblem(p)
    out = torch.full((p.colidx.size,), float("nan"), device="cuda:0")
    ws = torch.empty(binding.sgap_sddmm_csr_workspace_size(p.K, p.N, window_kb), dtype=torch.uint8, device="cuda:0")
    binding.sgap_sddmm_csr_windows(p.M, p.K, p.N, dp.rowptr, dp.colidx, dp.vals, torch.from_numpy(X1).cuda(), dp.B, out, 8,
                                   binding.STRATEGIES["parallel"], min_len, window_kb, workspace=ws)
    torch.cuda.synchronize()
    assert ws.view(torch.int32)[LDS_RUNS].item() == runs, f"{what}: the other kernel"
    got = out.cpu().numpy().astype(np.float64)
    assert not np.isnan(got).any(), f"{what}: entries left unwritten"
    bad = got != ref if exact else np.abs(got - ref) > TOL * bnd
    assert not bad.any(), f"{what}: {bad.sum()} entries off, the first is {np.flatnonzero(bad)[0]}"


# 64 columns are one tile; 68 and 100 two of which lanes stay idle.  4,768 columns: shares of 596 for 8 dies
@pytest.mark.parametrize("J", [64, 68, 100, 128, 192, 252, 256])
@pytest.mark.parametrize("K", [700, 4767, 4769])
def test_columns_and_windows(J, K):
    p = problem(300, K, J, min(600, K // 2), seed=J + K)
    for window_kb in (149, 64, 1):  # 596, 256 and 4 columns
        check(p, 40, f"J={J} K={K} {window_kb} KiB", window_kb=window_kb)


# the lengths are ranked 2,048 at a time; the workspace has room for 8,192 rows' pointers of 3 windows, 32,768, of which every row
# needs nine (the shares of 8 dies)
@pytest.mark.parametrize("n_long,runs", [(255, 0), (256, 1), (257, 1), (1279, 1), (1281, 1), (2048, 1), (2049, 1), (3640, 1), (3641, 0)])
def test_rows(n_long, runs):
    check(problem(n_long, 1500, 64, 160, seed=n_long), 30, f"{n_long} rows", runs=runs)


# 7 to 9, 15 to 17, 31 to 33 and many entries in a window
@pytest.mark.parametrize("longest,K", [(7, 56), (8, 56), (9, 56), (15, 120), (16, 120), (17, 120), (24, 180), (25, 180),
                                       (31, 240), (32, 240), (33, 240), (120, 120), (600, 600), (4700, 4768)])
def test_entries_of_a_window(longest, K):
    check(problem(260, K, 64, longest, seed=longest, shortest=longest), longest, f"{longest} of {K}")


@pytest.mark.parametrize("n_long", [300, 1300])
def test_unsorted_and_repeated_columns(n_long):
    p = problem(n_long, 4000, 68, 500, seed=n_long)
    rng = np.random.default_rng(7)
    for i in range(p.M):
        a, b = p.rowptr[i], p.rowptr[i + 1]
        if i % 3 == 0:
            perm = rng.permutation(b - a)
            p.colidx[a:b], p.vals[a:b] = p.colidx[a:b][perm], p.vals[a:b][perm]
        elif b - a > 20:
            j = a + int(rng.integers(b - a - 1))
            p.colidx[j], p.colidx[j + 1] = p.colidx[j + 1], p.colidx[j]
            p.colidx[a + 3] = p.colidx[a + 2]
    check(p, 60, "unsorted")
    check(p, 60, "unsorted, many windows", window_kb=16)


# rows of one length, which the list holds in any order, a third of them without order of the columns
@pytest.mark.parametrize("J", [68, 256])
def test_the_rows_beside_a_row_do_not_change_its_results(J):
    M, K, length = 600, 3000, 400
    rng = np.random.default_rng(J)
    cols = np.sort(rng.permuted(np.tile(np.arange(K, dtype=np.int32), (M, 1)), axis=1)[:, :length], axis=1)
    cols[::3] = rng.permuted(cols[::3], axis=1)
    vals, X1 = (wl.fill_values(rng, M * n, False).reshape(M, n) for n in (length, J))
    rowptr = np.arange(M + 1, dtype=np.int32) * length

    def run(order):
        p = wl.SpmmProblem("order", M, K, J, rowptr, cols[order].ravel(), vals[order].ravel(), B)
        X1d = torch.from_numpy(X1[order]).cuda()
        return DeviceProblem(p).run_sddmm_windows(X1d, 8, "parallel", length, 149).cpu().numpy().reshape(M, length)

    B = wl.fill_values(rng, K * J, False).reshape(K, J)
    first = run(np.arange(M))
    for order in (np.arange(M)[::-1], rng.permutation(M)):
        assert np.array_equal(run(order), first[order])


def test_infinite_and_nan_rows_reach_only_the_entries_that_name_them():
    p = problem(400, 3000, 68, 300, seed=5)
    p.B[11], p.B[1500], p.B[2999] = np.inf, np.nan, -np.inf
    X1 = np.abs(wl.fill_values(np.random.default_rng(1), p.M * p.N, False).reshape(p.M, p.N)) + 1
    dp = DeviceProblem(p)
    got = dp.run_sddmm_windows(torch.from_numpy(X1.astype(np.float32)).cuda(), 8, "parallel", 40, 149).cpu().numpy()
    named = np.isin(p.colidx, (11, 1500, 2999))
    assert np.isfinite(got[~named]).all()
    with np.errstate(invalid="ignore"):
        assert np.array_equal(got[named], p.vals[named] * p.B[p.colidx[named], 0], equal_nan=True)


def test_floats_where_the_rule_takes_it():
    check(problem(300, 26000, 128, 3000, seed=9, integer=False), 500, "floats", exact=False, window_kb=0)


def test_the_size_of_the_windows_chooses_between_lds_and_the_l2():
    p = problem(300, 26000, 128, 3000, seed=11)
    for window_kb, runs in ((0, 1), (149, 1), (150, 0), (2048, 0)):
        check(p, 500, f"{window_kb} KiB", window_kb=window_kb, runs=runs)


@pytest.mark.parametrize("shape", [without_order, crowded])
def test_rows_that_windows_in_lds_would_not_serve(shape):
    args = (300, 26000, 128, 3000)
    long = np.flatnonzero(np.diff(problem(*args, seed=12).rowptr) > 500)
    assert long.size == 300
    for rows, runs in ((long, 0), (long[::4], 0), (long[:0], 1)):
        check(shape(problem(*args, seed=12), rows), 500, f"{rows.size} rows", window_kb=0, runs=runs)


def test_rows_too_thin_for_it():
    check(problem(700, 20000, 256, 200, seed=10), 40, "thin", window_kb=0, runs=0)


def test_a_few_rows_far_denser_than_the_others():
    p = problem(600, 9000, 64, 90, seed=3)
    rng = np.random.default_rng(4)
    lengths = np.diff(p.rowptr)
    long = np.flatnonzero(lengths > 30)
    lengths[long[5]], lengths[long[300]] = 8900, 4000
    rowptr, colidx = wl.csr_from_lengths(rng, lengths, p.K)
    check(wl.SpmmProblem("dense rows", p.M, p.K, p.N, rowptr, colidx, wl.fill_values(rng, colidx.size, True), p.B), 20, "dense rows")


@pytest.mark.parametrize("J", [64, 128])
def test_the_row_behind_a_long_one(J):
    rng = np.random.default_rng(J)
    M, K = 1200, 700
    lengths = np.where(np.arange(M) % 2 == 0, rng.integers(100, 350, M), 1)
    rowptr, colidx = wl.csr_from_lengths(rng, lengths, K)
    behind = rowptr[1:-1:2]
    colidx[behind] = rng.integers(K - 20, K, behind.size)
    p = wl.SpmmProblem("behind", M, K, J, rowptr, colidx, wl.fill_values(rng, colidx.size, True),
                       wl.fill_values(rng, K * J, True).reshape(K, J))
    check(p, 90, f"J={J}")
