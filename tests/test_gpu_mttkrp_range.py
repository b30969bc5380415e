"""MTTKRP multiplies an entry with its row of X2 first and the row of X1 last (the fiber's sum comes before the factor of
the fiber): values that meet in range in that order, and only in that order, give the exact result at every point.  Where
stored entries are the unit of work a fiber that a tile or a lane's share cuts is multiplied part by part; the fibers of the first
test are too short for that to matter."""
import numpy as np
import pytest
import torch

import oracle
from paper_2209_02882_amd import binding
from paper_2209_02882_amd import workloads as wl
from paper_2209_02882_amd.device import DeviceTensor3

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("up", [100, -100])
@pytest.mark.parametrize("J", [3, 20, 32])
def test_no_product_leaves_the_range(J, up):
    t = wl.make_tensor3("tensor3_small_int", J=J)
    ref, _ = oracle.mttkrp_csf(t.I, t.K, t.L, t.J, t.fptr, t.fidx, t.eptr, t.eidx, t.vals, t.X1, t.X2)
    # integers times powers of two: vals * X2 stays small, vals * X1 is 2^200 or 2^-200 of it; the sums are exact as ever
    scale = np.float32(2.0) ** np.float32(up)
    t.vals, t.X1, t.X2 = t.vals * scale, t.X1 * scale, t.X2 / scale
    dt = DeviceTensor3(t)
    for g in binding.GROUP_SIZES:
        for strategy in binding.STRATEGIES:
            for schedule in binding.SCHEDULES:
                got = dt.run_mttkrp(g, strategy, schedule).cpu().numpy().astype(np.float64)
                assert np.array_equal(got, ref * 2.0 ** up), (g, strategy, schedule)


LENGTHS = [1, 40, 33, 64, 300, 0, 7, 2000, 3300, 3400, 96, 500, 0]  # of fibers: some that several teams of lanes share, one that a block has no room for


@pytest.mark.parametrize("J", [1, 3, 20, 32, 70])
def test_a_fiber_is_summed_whole_whatever_its_length(J):
    """Slices as the unit of work: the parts of a long fiber meet before the row of X1 multiplies them.  Parts of +-2^10 and more and a
    row of X1 of 2^118 would leave the range, a part that is zero would make an infinity NaN."""
    rng = np.random.default_rng(J)
    slices, L = 37, 4000
    fptr, fidx = wl.csr_from_lengths(rng, rng.integers(0, 4, slices), 50)
    eptr, eidx = wl.csr_from_lengths(rng, np.resize(LENGTHS, fidx.size), L)
    X1 = np.full((50, J), 2.0**118, np.float32)
    X2 = np.ones((L, J), np.float32)
    vals = np.zeros(eidx.size, np.float32)
    t = np.zeros(fidx.size)
    X1[::7] = np.inf
    for f, (a, b) in enumerate(zip(eptr, eptr[1:])):
        if b - a < 2:
            vals[a:b] = t[f] = 1 if b > a else 0
            continue
        if X1[fidx[f], 0] == np.inf:  # nothing in the first half
            vals[(a + b) // 2:b] = 1
            t[f] = b - (a + b) // 2
        else:
            half = (b - a) // 2
            vals[a:a + half], vals[a + half:a + 2 * half] = 2.0**10, -2.0**10
            vals[b - 1] += 0 if (b - a) % 2 == 0 else 3
            t[f] = 0 if (b - a) % 2 == 0 else 3
    with np.errstate(invalid="ignore"):
        product = X1[fidx, :1].astype(np.float64) * t[:, None]
    ref = np.zeros((slices, 1))
    for i, (a, b) in enumerate(zip(fptr, fptr[1:])):
        ref[i] = product[a:b].sum(0)
    d = [torch.from_numpy(x).cuda() for x in (fptr, fidx, eptr, eidx, vals, X1, X2)]
    for strategy in binding.STRATEGIES.values():
        for g in (1, 8, 64):
            for hint in (-1, eidx.size, 10**9):
                Y = torch.empty((slices, J), device="cuda")
                binding.sgap_mttkrp_csf_ex(slices, 50, L, J, *d, Y, g, strategy, binding.SGAP_SCHED_ROW_SPLIT, nnz_hint=hint)
                got = Y.cpu().numpy().astype(np.float64)
                assert np.array_equal(got, np.broadcast_to(ref, got.shape), equal_nan=True), (strategy, g, hint)


@pytest.mark.parametrize("J", [1, 3, 8, 20, 32, 70])
def test_fibers_without_entries_have_no_part_where_entries_are_the_unit_of_work(J):
    """X1 is not finite in the rows that only such fibers name.  They lie amid a tile, at its ends, and many in a row."""
    rng = np.random.default_rng(J)
    slices, K, L = 1200, 64, 500
    fptr, fidx = wl.csr_from_lengths(rng, rng.integers(0, 25, slices), K)
    eptr, eidx = wl.csr_from_lengths(rng, np.where(fidx % 2 == 0, 0, np.resize([1, 3, 1, 40, 2, 8], fidx.size)), L)
    vals = wl.fill_values(rng, eidx.size, True)
    X1, X2 = (wl.fill_values(rng, n * J, True).reshape(n, J) for n in (K, L))
    X1[::2] = 0
    ref, _ = oracle.mttkrp_csf(slices, K, L, J, fptr, fidx, eptr, eidx, vals, X1, X2)
    X1[::4], X1[2::4] = np.inf, np.nan
    d = [torch.from_numpy(x).cuda() for x in (fptr, fidx, eptr, eidx, vals, X1, X2)]
    for strategy in binding.STRATEGIES.values():
        for g in (1, 8, 64):
            for hint in (-1, eidx.size, 10**9):
                Y = torch.empty((slices, J), device="cuda")
                binding.sgap_mttkrp_csf_ex(slices, K, L, J, *d, Y, g, strategy, binding.SGAP_SCHED_NNZ_BALANCED, nnz_hint=hint)
                assert np.array_equal(Y.cpu().numpy().astype(np.float64), ref), (strategy, g, hint)
