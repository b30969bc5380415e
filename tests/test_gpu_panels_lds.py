"""Long rows whose windows of B lie in LDS (lists of at least 256 long rows, N >= 64): exact on integer-valued inputs, at the
edges of teams, slots, column tiles, windows and shares.  A window_kb of at most 154 asks for these windows at any size."""
import numpy as np
import pytest
import torch

from paper_2209_02882_amd import binding
from paper_2209_02882_amd import workloads as wl

from gpu_util import DeviceProblem, assert_close, full_reference
from test_window_form import plan

pytestmark = pytest.mark.gpu

LDS_RUNS = 19  # place of the word of the workspace that says whether the LDS kernel runs


def problem(n_long, K, N, longest, seed, shortest=None, integer=True):
    """n_long long rows among four times as many short ones."""
    rng = np.random.default_rng(seed)
    M = 5 * n_long + 3
    lengths = rng.integers(0, 6, M)
    at = rng.choice(M, n_long, replace=False)
    lengths[at] = rng.integers(longest // 4 if shortest is None else shortest, longest + 1, n_long)
    rowptr, colidx = wl.csr_from_lengths(rng, lengths, K)
    return wl.SpmmProblem("lds", M, K, N, rowptr, colidx, wl.fill_values(rng, colidx.size, integer),
                          wl.fill_values(rng, K * N, integer).reshape(K, N))


def check(p, min_len, what, exact=True, window_kb=154, runs=1, points=((1, "serial"), (4, "parallel"))):
    dp = DeviceProblem(p)
    C_ref, BND = full_reference(p)
    for g, st in points:
        cfg = binding.make_config(g, st, "row_split", long_row_min=min_len, window_kb=window_kb)
        ws, C = dp.workspace_for(cfg), dp.new_output(poison=True)
        dp.launch_cfg(C, cfg, ws)
        torch.cuda.synchronize()
        assert ws.view(torch.int32)[LDS_RUNS].item() == runs, f"{what}: the other kernel"
        assert_close(C, C_ref, BND, exact=exact, what=f"{what} {g} {st}")


# 64 columns are one tile; 68 and 100 two of which lanes stay idle; 260 five.  5,088 columns: shares of 636 for 8 dies
@pytest.mark.parametrize("N", [64, 68, 100, 128, 192, 256, 260])
@pytest.mark.parametrize("K", [700, 5087, 5089])
def test_columns_and_windows(N, K):
    p = problem(300, K, N, min(600, K // 2), seed=N + K)
    for window_kb in (154, 64, 1):  # 616, 256 and 4 columns
        check(p, 40, f"N={N} K={K} {window_kb} KiB", window_kb=window_kb, points=[(1, "serial")])


# rows of a wavefront's teams, of a slot, of a workgroup (1,280) and of two: one fewer, one more
@pytest.mark.parametrize("n_long,runs", [(255, 0), (256, 1), (257, 1), (1279, 1), (1281, 1), (2563, 1)])
def test_rows(n_long, runs):
    check(problem(n_long, 1500, 64, 160, seed=n_long), 30, f"{n_long} rows", runs=runs)


# 15 to 17, 31 to 33 and many entries in a window; every column of the window in a row
@pytest.mark.parametrize("longest,K", [(15, 120), (16, 120), (17, 120), (31, 240), (33, 240), (120, 120), (600, 600), (4800, 4928)])
def test_entries_of_a_window(longest, K):
    check(problem(260, K, 64, longest, seed=longest, shortest=longest), longest, f"{longest} of {K}")


@pytest.mark.parametrize("n_long", [300, 1300])
def test_unsorted_and_repeated_columns(n_long):
    p = problem(n_long, 4000, 68, 500, seed=n_long)
    rng = np.random.default_rng(7)
    for i in range(p.M):
        a, b = p.rowptr[i], p.rowptr[i + 1]
        if i % 3 == 0:  # all of the row, or two neighbours of it, out of order
            perm = rng.permutation(b - a)
            p.colidx[a:b], p.vals[a:b] = p.colidx[a:b][perm], p.vals[a:b][perm]
        elif b - a > 20:
            j = a + int(rng.integers(b - a - 1))
            p.colidx[j], p.colidx[j + 1] = p.colidx[j + 1], p.colidx[j]
            p.colidx[a + 3] = p.colidx[a + 2]
    check(p, 60, "unsorted")
    check(p, 60, "unsorted, many windows", window_kb=16)


def test_infinite_and_nan_rows_of_b_reach_only_the_rows_that_name_them():
    p = problem(400, 3000, 64, 300, seed=5)
    p.B[11], p.B[1500], p.B[2999] = np.inf, np.nan, -np.inf
    dp = DeviceProblem(p)
    cfg = binding.make_config(1, "serial", "row_split", long_row_min=40, window_kb=154)
    got = dp.run_cfg(cfg).cpu().numpy()
    named = np.array([np.isin(p.colidx[a:b], (11, 1500, 2999)).any() for a, b in zip(p.rowptr[:-1], p.rowptr[1:])])
    assert np.isfinite(got[~named]).all() and not np.isfinite(got[named]).any()


def test_floats_where_the_rule_takes_it():
    check(problem(1300, 9000, 128, 6000, seed=9, integer=False), 500, "floats", exact=False, window_kb=0)


# (which the tests of test_window_form.py rest on)
@pytest.mark.parametrize("n_long,K,N,longest", [(260, 9000, 64, 3000), (1300, 9000, 128, 6000), (700, 20000, 160, 4000), (300, 5000, 260, 700)])
def test_the_device_chooses_as_the_host_does(n_long, K, N, longest):
    p = problem(n_long, K, N, longest, seed=n_long, shortest=longest // 3)
    dp = DeviceProblem(p)
    lengths = np.diff(p.rowptr)
    long = lengths[lengths >= longest // 4]
    cfg = binding.make_config(1, "serial", "row_split", long_row_min=longest // 4)
    ws = dp.workspace_for(cfg)
    dp.launch_cfg(dp.new_output(), cfg, ws)
    head = ws[:256].view(torch.int32).cpu().tolist()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    on, groups, shares, window, _, _ = plan("spmm", K, N, long.size, int(long.sum()), int(long.max()), int(p.rowptr[-1]),
                                            head[28], head[27], cus=cus)
    assert head[0] == long.size and head[16] == long.sum() and head[30] == long.max()
    assert head[LDS_RUNS] == on and (not on or (head[22], head[24], head[26]) == (groups, shares, window))


def test_the_size_of_the_windows_chooses_between_lds_and_the_l2():
    p = problem(1300, 9000, 128, 6000, seed=11)
    for window_kb, runs in ((0, 1), (154, 1), (155, 0), (3072, 0)):
        check(p, 500, f"{window_kb} KiB", window_kb=window_kb, runs=runs)


def without_order(p, rows):
    """p with the entries of these rows in any order."""
    rng = np.random.default_rng(1)
    for i in rows:
        a, b = p.rowptr[i], p.rowptr[i + 1]
        perm = rng.permutation(b - a)
        p.colidx[a:b], p.vals[a:b] = p.colidx[a:b][perm], p.vals[a:b][perm]
    return p


def crowded(p, rows):
    """p with the entries of these rows side by side, somewhere."""
    rng = np.random.default_rng(1)
    for i in rows:
        a, b = p.rowptr[i], p.rowptr[i + 1]
        p.colidx[a:b] = rng.integers(p.K - (b - a) + 1) + np.arange(b - a)
    return p


# the windows in LDS serve rows whose columns ascend and lie apart; the others, and lists with some of them, are gathered
@pytest.mark.parametrize("shape", [without_order, crowded])
def test_rows_that_windows_in_lds_would_not_serve(shape):
    n_long, args = 1300, (1300, 9000, 128, 6000)
    long = np.flatnonzero(np.diff(problem(*args, seed=12).rowptr) > 500)
    assert long.size == n_long
    for rows, runs in ((long, 0), (long[::4], 0), (long[:0], 1)):
        check(shape(problem(*args, seed=12), rows), 500, f"{rows.size} rows", window_kb=0, runs=runs)


def test_rows_too_thin_for_it():
    check(problem(700, 20000, 64, 200, seed=10), 40, "thin", window_kb=0, runs=0)


# one row of nearly every column among rows of few: more than the 32 entries a slot takes at once, in most windows
def test_a_few_rows_far_denser_than_the_others():
    p = problem(600, 9000, 64, 90, seed=3)
    rng = np.random.default_rng(4)
    lengths = np.diff(p.rowptr)
    long = np.flatnonzero(lengths > 30)
    lengths[long[5]], lengths[long[300]] = 8900, 4000
    rowptr, colidx = wl.csr_from_lengths(rng, lengths, p.K)
    q = wl.SpmmProblem("dense rows", p.M, p.K, p.N, rowptr, colidx, wl.fill_values(rng, colidx.size, True), p.B)
    check(q, 20, "dense rows")


# a short row behind a long one whose column lies where the long one's last entries do
@pytest.mark.parametrize("N", [64, 128])
def test_the_row_behind_a_long_one(N):
    rng = np.random.default_rng(N)
    M, K = 1200, 700
    lengths = np.where(np.arange(M) % 2 == 0, rng.integers(100, 350, M), 1)
    rowptr, colidx = wl.csr_from_lengths(rng, lengths, K)
    behind = rowptr[1:-1:2]
    colidx[behind] = rng.integers(K - 20, K, behind.size)
    p = wl.SpmmProblem("behind", M, K, N, rowptr, colidx, wl.fill_values(rng, colidx.size, True),
                       wl.fill_values(rng, K * N, True).reshape(K, N))
    check(p, 90, f"N={N}")
