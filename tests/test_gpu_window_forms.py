"""The forms that long rows by column windows have (windows in LDS, owner wavefronts, wavefronts that claim pieces), each where
it has more than one pass, job or window to do: exact on integer-valued inputs, and which form ran."""
import numpy as np
import pytest
import torch

import oracle
from paper_2209_02882_amd import binding
from paper_2209_02882_amd import workloads as wl

from gpu_util import DeviceProblem, assert_close, full_reference
from test_gpu_panels_lds import problem, without_order

pytestmark = pytest.mark.gpu

ROWS, CLAIMED, IN_LDS, TILES, GROUPS, SHARES = 0, slice(1, 9), 19, 20, 22, 24  # words of the workspace


def header(ws):
    return ws[:256].view(torch.int32).cpu().numpy()


def form(ws):
    head = header(ws)
    return "lds" if head[IN_LDS] else "claims" if head[CLAIMED].any() else "owners" if head[ROWS] >= 256 else "none"


def spmm(p, min_len, window_kb, wanted, max_long_rows=0, points=((1, "serial"), (4, "parallel"))):
    dp = DeviceProblem(p)
    C_ref, BND = full_reference(p)
    for g, st in points:
        cfg = binding.make_config(g, st, "row_split", long_row_min=min_len, window_kb=window_kb, max_long_rows=max_long_rows)
        ws, C = dp.workspace_for(cfg), dp.new_output(poison=True)
        dp.launch_cfg(C, cfg, ws)
        torch.cuda.synchronize()
        assert form(ws) == wanted
        assert_close(C, C_ref, BND, exact=True, what=f"{wanted} {g} {st}")
    return header(ws)


def sddmm(p, min_len, window_kb, wanted, max_long_rows=0):
    X1 = wl.fill_values(np.random.default_rng(p.M), p.M * p.N, True).reshape(p.M, p.N)
    ref, _ = oracle.sddmm_csr(p.M, p.K, p.N, p.rowptr, p.colidx, p.vals, X1, p.B, nthreads=8, bound=False)
    dp = DeviceProblem(p)
    out = torch.full((p.colidx.size,), float("nan"), device="cuda:0")
    ws = torch.empty(binding.sgap_sddmm_csr_workspace_size(p.K, p.N, window_kb, max_long_rows), dtype=torch.uint8, device="cuda:0")
    binding.sgap_sddmm_csr_windows(p.M, p.K, p.N, dp.rowptr, dp.colidx, dp.vals, torch.from_numpy(X1).cuda(), dp.B, out, 8,
                                   binding.STRATEGIES["parallel"], min_len, window_kb, max_long_rows, workspace=ws)
    torch.cuda.synchronize()
    assert form(ws) == wanted
    assert np.array_equal(out.cpu().numpy().astype(np.float64), ref)
    return header(ws)


def thin(n_long, N, seed):
    """Long rows of 40 to 160 entries, every third without order and with repeated columns; nine windows of 160 KiB per die at
    N = 256."""
    p = problem(n_long, 12000, N, 160, seed=seed)
    p = without_order(p, range(0, p.M, 3))
    long = np.flatnonzero(np.diff(p.rowptr) >= 40)[::3]
    p.colidx[p.rowptr[long] + 7] = p.colidx[p.rowptr[long] + 5]
    return p


# 5,300 rows: more than the 5,120 that the wavefronts of a die own in one pass.  260 and 512 columns: two tiles
@pytest.mark.parametrize("N,n_long", [(132, 700), (200, 5300), (256, 700), (256, 5300), (260, 700), (512, 700)])
def test_owner_wavefronts(N, n_long):
    spmm(thin(n_long, N, N + n_long), 40, 160, "owners")


@pytest.mark.parametrize("J,n_long", [(132, 700), (200, 5300), (252, 700), (256, 5300)])
def test_owner_wavefronts_of_sddmm(J, n_long):
    sddmm(thin(n_long, J, J + n_long), 40, 160, "owners")


@pytest.mark.parametrize("N,n_long", [(64, 700), (128, 700), (256, 200)])
def test_claiming_wavefronts(N, n_long):
    spmm(thin(n_long, N, N), 40, 160, "claims")
    sddmm(thin(n_long, N, N), 40, 160, "claims")


def test_owner_wavefronts_with_offsets_of_64_bits():
    K, N, M, n_long = 1 << 22, 256, 900, 300  # K * N * 4 = 2^32
    rng = np.random.default_rng(5)
    lengths = rng.integers(0, 12, M)
    lengths[::3] = rng.integers(300, 1200, n_long)
    rowptr, colidx = wl.csr_from_lengths(rng, lengths, K)
    colidx[rowptr[M - 3 + 1] - 1] = K - 1  # the far end of B is touched
    vals = wl.fill_values(rng, colidx.size, True)
    used = np.unique(colidx)
    B_used = wl.fill_values(rng, used.size * N, True).reshape(-1, N)
    B = torch.zeros((K, N), device="cuda:0")
    B[torch.from_numpy(used.astype(np.int64)).cuda()] = torch.from_numpy(B_used).cuda()
    at = np.searchsorted(used, colidx).astype(np.int32)  # the same rows of B by their place among those that are used
    rp, ci, va = (torch.from_numpy(x).cuda() for x in (rowptr, colidx, vals))
    C_ref, BND = oracle.spmm_csr(M, used.size, N, rowptr, at, vals, B_used)
    C = torch.full((M, N), float("nan"), device="cuda:0")
    cfg = binding.make_config(1, "serial", "row_split", long_row_min=300, window_kb=3072)
    ws = torch.empty(binding.sgap_spmm_csr_workspace_size(M, K, N, cfg), dtype=torch.uint8, device="cuda:0")
    binding.sgap_spmm_csr_cfg(M, K, N, rp, ci, va, B, C, cfg, workspace=ws)
    torch.cuda.synchronize()
    assert form(ws) == "owners"
    assert_close(C, C_ref, BND, exact=True)
    X1 = wl.fill_values(rng, M * N, True).reshape(M, N)
    ref, _ = oracle.sddmm_csr(M, used.size, N, rowptr, at, vals, X1, B_used, nthreads=8, bound=False)
    out = torch.full((colidx.size,), float("nan"), device="cuda:0")
    ws = torch.empty(binding.sgap_sddmm_csr_workspace_size(K, N, 2048), dtype=torch.uint8, device="cuda:0")
    binding.sgap_sddmm_csr_windows(M, K, N, rp, ci, va, torch.from_numpy(X1).cuda(), B, out, 8, binding.STRATEGIES["parallel"], 300,
                                   2048, workspace=ws)
    torch.cuda.synchronize()
    assert form(ws) == "owners"
    assert np.array_equal(out.cpu().numpy().astype(np.float64), ref)


# a workgroup's second job: 33 tiles of columns for 32 workgroups, and (SDDMM) 34 groups of rows
def test_more_jobs_than_workgroups():
    head = spmm(problem(300, 1000, 2112, 100, seed=1), 25, 154, "lds", points=[(1, "serial")])
    assert head[TILES] * head[GROUPS] * head[SHARES] > 32
    head = sddmm(problem(43_000, 300, 64, 12, seed=2, shortest=8), 8, 149, "lds", max_long_rows=1 << 18)
    assert head[GROUPS] * head[SHARES] > 32


# a list of more than 8,192 rows is in the order of finding
def test_lists_that_are_not_sorted():
    p = problem(9000, 1000, 128, 40, seed=3, shortest=30)
    spmm(p, 30, 154, "lds", max_long_rows=16384, points=[(1, "serial")])
    sddmm(problem(9000, 5000, 64, 40, seed=4, shortest=30), 30, 149, "lds", max_long_rows=16384)


# captured once, replayed on columns in order and without: what the header of the workspace holds from the replay before
# (among it the longest row and what windows in LDS would not serve) decides nothing
@pytest.mark.parametrize("N,gathering", [(160, "owners"), (128, "claims")])
def test_a_graph_replayed_on_other_columns(N, gathering):
    p = problem(1300, 9000, N, 6000, seed=N)
    order = p.colidx.copy(), p.vals.copy()
    without_order(p, range(p.M))
    orders = {"lds": order, gathering: (p.colidx, p.vals)}
    C_ref, BND = full_reference(p)
    X1 = wl.fill_values(np.random.default_rng(N), p.M * N, True).reshape(p.M, N)
    X1d, dp = torch.from_numpy(X1).cuda(), DeviceProblem(p)
    cfg = binding.make_config(1, "serial", "row_split", long_row_min=1500)
    ws, C = dp.workspace_for(cfg), dp.new_output()
    ws2 = torch.empty(binding.sgap_sddmm_csr_workspace_size(p.K, N), dtype=torch.uint8, device="cuda:0")
    out = torch.empty(p.colidx.size, device="cuda:0")

    def calls():
        dp.launch_cfg(C, cfg, ws, stream=torch.cuda.current_stream())
        binding.sgap_sddmm_csr_windows(p.M, p.K, N, dp.rowptr, dp.colidx, dp.vals, X1d, dp.B, out, 8, binding.STRATEGIES["parallel"],
                                       1500, workspace=ws2, stream=torch.cuda.current_stream())

    calls()  # eager, once per kernel
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        calls()
    for wanted in ("lds", gathering, "lds", "lds", gathering):
        colidx, vals = orders[wanted]
        dp.colidx.copy_(torch.from_numpy(colidx))
        dp.vals.copy_(torch.from_numpy(vals))
        C.fill_(float("nan"))
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert (form(ws), form(ws2)) == (wanted, wanted)
        assert_close(C, C_ref, BND, exact=True, what=wanted)
        ref, _ = oracle.sddmm_csr(p.M, p.K, N, p.rowptr, colidx, vals, X1, p.B, nthreads=8, bound=False)
        assert np.array_equal(out.cpu().numpy().astype(np.float64), ref), wanted
