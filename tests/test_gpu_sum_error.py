"""How far sums are from 64 bits where teams of lanes go through a row (or a slice) at their own pace, against the orders that the point
of the design space is described with: a group's members with a share each, whose sums meet in a tree (parallel), and group_size
consecutive entries in a chain, whose sums are added up in order (serial).  The other orders are written out here in fp32.

The bound: the rounding errors of a sum of random signs have a variance in proportion to the terms behind each partial sum.  Batches
of eight as a tree, in two chains that take turns, have at most 124/120 of a group of eight's (rows of 24), a slice's fibers in four
chains 768/720 (24 fibers of four entries): 1.7 and 3.3 % in the root mean square; and 200,000 sums of each kind leave 0.5 %."""
import numpy as np
import pytest
import torch

from paper_2209_02882_amd import binding
from paper_2209_02882_amd import workloads as wl

pytestmark = pytest.mark.gpu

MOST = 1.04


def uniform(rng, *shape):
    return rng.uniform(-1, 1, shape).astype(np.float32)


def fma(a, b, c):
    """fp32: the product is exact in 64 bits."""
    return (a.astype(np.float64) * b + c).astype(np.float32)


def tree(parts):
    """Pairwise over the first axis (a power of two)."""
    while len(parts) > 1:
        parts = parts[:len(parts) // 2] + parts[len(parts) // 2:]
    return parts[0]


def rms(got, exact):
    return np.sqrt(np.mean((got.astype(np.float64) - exact) ** 2))


def spmm_rows(rng, length, n, columns):
    """A matrix one row in eight of which has `length` entries, the others few, and what those rows multiply: values and rows of B
    with an axis of their own for the entries."""
    rows = 48_000
    lengths = rng.integers(8, 13, rows)
    lengths[::8] = length
    rowptr, colidx = wl.csr_from_lengths(rng, lengths, columns)
    vals, B = uniform(rng, colidx.size), uniform(rng, columns, n)
    at = rowptr[:-1][::8, None] + np.arange(length)
    return rowptr, colidx, vals, B, at, vals[at].T[:, :, None], B[colidx[at]].transpose(1, 0, 2)


def spmm(rowptr, colidx, vals, B, g, strategy, schedule):
    m, (k, n) = rowptr.size - 1, B.shape
    C = torch.empty((m, n), device="cuda")
    binding.sgap_spmm_csr_ex(m, k, n, *(torch.from_numpy(x).cuda() for x in (rowptr, colidx, vals, B)), C, g, strategy, schedule,
                             nnz_hint=colidx.size)
    return C.cpu().numpy()[::8]


@pytest.mark.parametrize("length", [8, 16, 24, 32, 64, 90])
def test_row_split_parallel(length):
    rng = np.random.default_rng(length)
    n = 32
    rowptr, colidx, vals, B, _, v, b = spmm_rows(rng, length, n, 5000)
    exact = (v.astype(np.float64) * b).sum(0)
    for g in (8, 16, 32):
        members = np.zeros((g, *exact.shape), np.float32)
        for e in range(length):
            members[e % g] = fma(v[e], b[e], members[e % g])
        got = spmm(rowptr, colidx, vals, B, g, binding.SGAP_REDUCE_PARALLEL, binding.SGAP_SCHED_ROW_SPLIT)
        print(f"  row-split parallel, rows of {length}, G = {g}: {rms(got, exact):.3e}, group by group {rms(tree(members), exact):.3e}")
        assert rms(got, exact) <= MOST * rms(tree(members), exact), g


@pytest.mark.parametrize("n", [32, 64])
@pytest.mark.parametrize("length", [8, 16, 32, 64, 90])
def test_nnz_balanced_serial(length, n):
    rng = np.random.default_rng(length)
    rowptr, colidx, vals, B, at, v, b = spmm_rows(rng, length, n, 5000)
    exact = (v.astype(np.float64) * b).sum(0)
    for g in (8, 16, 32):
        total, share = np.zeros(exact.shape, np.float32), np.zeros(exact.shape, np.float32)
        for e in range(length):
            ends = ((at[:, e] + 1) % g == 0)[:, None]  # of a lane's entries
            share = fma(v[e], b[e], share)
            total = np.where(ends, total + share, total)
            share = np.where(ends, np.float32(0), share)
        total = total + share
        got = spmm(rowptr, colidx, vals, B, g, binding.SGAP_REDUCE_SERIAL, binding.SGAP_SCHED_NNZ_BALANCED)
        print(f"  nnz-balanced serial, rows of {length}, N = {n}, G = {g}: {rms(got, exact):.3e}, lane by lane {rms(total, exact):.3e}")
        assert rms(got, exact) <= MOST * rms(total, exact), g


@pytest.mark.parametrize("fibers,entries", [(2, 16), (4, 4), (8, 4), (8, 9), (16, 4), (24, 4)])
def test_mttkrp_by_slices(fibers, entries):
    rng = np.random.default_rng(fibers * entries)
    slices, extent, j = 10_000, 2000, 32
    fptr, fidx = wl.csr_from_lengths(rng, np.full(slices, fibers), extent)
    eptr, eidx = wl.csr_from_lengths(rng, np.full(fidx.size, entries), extent)
    vals, X1, X2 = uniform(rng, eidx.size), uniform(rng, extent, j), uniform(rng, extent, j)
    shape = (slices, fibers, entries)
    v, x1, x2 = vals.reshape(shape), X1[fidx.reshape(shape[:2])], X2[eidx.reshape(shape)]
    exact = (x1.astype(np.float64) * (v[..., None].astype(np.float64) * x2).sum(2)).sum(1)
    t = np.zeros(x1.shape, np.float32)
    for e in range(entries):
        t = fma(v[:, :, e, None], x2[:, :, e], t)
    Y = torch.empty((slices, j), device="cuda")
    d = [torch.from_numpy(x).cuda() for x in (fptr, fidx, eptr, eidx, vals, X1, X2)]
    for g in (4, 8):
        members = np.zeros((g, *exact.shape), np.float32)
        for f in range(fibers):
            members[f % g] = fma(x1[:, f], t[:, f], members[f % g])
        binding.sgap_mttkrp_csf_ex(slices, extent, extent, j, *d, Y, g, binding.SGAP_REDUCE_PARALLEL, binding.SGAP_SCHED_ROW_SPLIT,
                                   nnz_hint=eidx.size)
        got = Y.cpu().numpy()
        print(f"  slices of {fibers} fibers of {entries}, G = {g}: {rms(got, exact):.3e}, group by group {rms(tree(members), exact):.3e}")
        assert rms(got, exact) <= MOST * rms(tree(members), exact), g
