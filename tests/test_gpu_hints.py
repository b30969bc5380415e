"""The caller's count of stored entries is a hint: whatever it says, every row of the result is written.  Exact on
integer-valued inputs, results poisoned with NaN before each call."""
import numpy as np
import pytest
import torch

import oracle
from paper_2209_02882_amd import binding
from paper_2209_02882_amd import workloads as wl

from gpu_util import POINTS, DeviceProblem

pytestmark = pytest.mark.gpu

# rows on both sides of the lengths from which a workgroup takes a row: max(256, 96 * G / passes over the columns)
LENGTHS = [0, 255, 256, 257, 3, 767, 768, 1000, 1536, 2047, 2048, 0, 1, 3072, 5000, 12] + [2] * 60 + [6144, 6]


def long_rows(N):
    rng = np.random.default_rng(N)
    K = 7000
    rowptr, colidx = wl.csr_from_lengths(rng, np.asarray(LENGTHS), K)
    p = wl.SpmmProblem("hints", len(LENGTHS), K, N, rowptr, colidx, wl.fill_values(rng, colidx.size, True),
                       wl.fill_values(rng, K * N, True).reshape(K, N))
    ref, _ = oracle.spmm_csr(p.M, p.K, p.N, p.rowptr, p.colidx, p.vals, p.B, nthreads=8, bound=False)
    return p, DeviceProblem(p), ref


@pytest.mark.parametrize("N", [1, 4, 37, 128, 300])
def test_row_split_with_any_hint(N):
    p, dp, ref = long_rows(N)
    C = dp.new_output()
    for hint in (0, 1, 100, 255, 256, p.nnz, 10 * p.nnz, -1):
        for g in binding.GROUP_SIZES:
            for strategy in ("parallel", "serial"):
                for knobs in ({}, {"persistent": 1}, {"tile_cols": 8, "rows_per_group": 3}):
                    C.fill_(float("nan"))
                    dp.launch_cfg(C, binding.make_config(g, strategy, "row_split", **knobs), nnz_hint=hint)
                    got = C.cpu().numpy().astype(np.float64)
                    assert np.array_equal(got, ref), (hint, g, strategy, knobs)


@pytest.mark.parametrize("N", [4, 37])
def test_the_other_paths_with_any_hint(N):
    p, dp, ref = long_rows(N)
    C = dp.new_output()
    for hint in (1, 100, 10 * p.nnz, -1):
        for point in POINTS:
            if point[2] == "nnz_balanced":
                got = dp.run(*point, C=C, nnz_hint=hint).cpu().numpy().astype(np.float64)
                assert np.array_equal(got, ref), (hint, point)
    X1 = wl.fill_values(np.random.default_rng(N), p.M * N, True).reshape(p.M, N)
    ref, _ = oracle.sddmm_csr(p.M, p.K, N, p.rowptr, p.colidx, p.vals, X1, p.B, nthreads=8, bound=False)
    X1d = torch.from_numpy(X1).cuda()
    out = torch.empty(p.nnz, device="cuda")
    for hint in (1, 100, 10 * p.nnz, -1):
        for g, strategy in ((1, "parallel"), (8, "parallel"), (64, "parallel"), (4, "serial")):
            out.fill_(float("nan"))
            dp.launch_sddmm(X1d, out, g, strategy, nnz_hint=hint)
            assert np.array_equal(out.cpu().numpy().astype(np.float64), ref), (hint, g, strategy)


def test_mttkrp_by_stored_entries_with_any_hint():
    t = wl.make_tensor3("tensor3_small_int")
    ref, _ = oracle.mttkrp_csf(t.I, t.K, t.L, t.J, t.fptr, t.fidx, t.eptr, t.eidx, t.vals, t.X1, t.X2)
    d = [torch.from_numpy(x).cuda() for x in (t.fptr, t.fidx, t.eptr, t.eidx, t.vals, t.X1, t.X2)]
    Y = torch.empty((t.I, t.J), device="cuda")
    for hint in (0, 1, 100, 10 * t.nnz, -1):
        for g in binding.GROUP_SIZES:
            for strategy in binding.STRATEGIES.values():
                Y.fill_(float("nan"))
                binding.sgap_mttkrp_csf_ex(t.I, t.K, t.L, t.J, *d, Y, g, strategy, binding.SGAP_SCHED_NNZ_BALANCED, nnz_hint=hint)
                assert np.array_equal(Y.cpu().numpy().astype(np.float64), ref), (hint, g, strategy)
