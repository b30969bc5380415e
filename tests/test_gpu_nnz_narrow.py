"""The segmented reduction of up to sixteen columns: rows that end at, before and behind the edges of a lane's entries, of a
wavefront, of a round of row pointers and of a tile (512 and 1,024 entries); exact on integer-valued inputs."""
import numpy as np
import pytest
import torch

import oracle
from paper_2209_02882_amd import binding
from paper_2209_02882_amd import workloads as wl

from gpu_util import DeviceProblem

pytestmark = pytest.mark.gpu


def rows_of(kind):
    if kind == "edges":  # of 8, 64, 256, 512, 1,024 and 2,048 entries
        at = sorted({e * i + d for e in (8, 64, 256, 512, 1024, 2048) for i in range(1, 4) for d in (-1, 0, 1)})
        return np.diff([0, *at, 7000])
    if kind == "one tile, full":
        return [1] * 2048
    if kind == "tiles of one row":
        return [1024, 2048, 4096, 1, 2047, 3, 6000]
    if kind == "runs without entries":  # in front, behind, and longer than a round of 256 and of 1,024 row pointers
        return [0] * 300 + [5] + [0] * 255 + [1] + [0] * 256 + [2] + [0] * 1024 + [9] + [0] * 5000 + [3000] + [0] * 1279 + [1] * 40 + [0] * 700
    if kind == "more tiles than a workgroup looks up or merges at once":
        return [600] * 470
    if kind == "short":
        return np.random.default_rng(1).integers(0, 4, 9001)
    return {"one entry": [1], "one row": [5000], "no entries": [0] * 900}[kind]


@pytest.mark.parametrize("kind", ["edges", "one tile, full", "tiles of one row", "runs without entries", "short", "one entry",
                                  "one row", "no entries", "more tiles than a workgroup looks up or merges at once"])
@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 13, 16, 17])
def test_rows_at_the_edges(N, kind):
    lengths = np.asarray(rows_of(kind))
    rng = np.random.default_rng(N)
    M, K = lengths.size, 6200
    rowptr, colidx = wl.csr_from_lengths(rng, lengths, K)
    p = wl.SpmmProblem("narrow", M, K, N, rowptr, colidx, wl.fill_values(rng, colidx.size, True),
                       wl.fill_values(rng, K * N, True).reshape(K, N))
    ref, _ = oracle.spmm_csr(p.M, p.K, p.N, p.rowptr, p.colidx, p.vals, p.B, nthreads=8, bound=False)
    dp = DeviceProblem(p)
    for hint in (colidx.size, min(1, colidx.size)):  # a workgroup per tile; one workgroup
        for g in (1, 16, 64):
            got = dp.run(g, "parallel", "nnz_balanced", nnz_hint=hint).cpu().numpy()
            assert np.array_equal(got.astype(np.float64), ref), (hint, g)


@pytest.mark.parametrize("N", [1, 4, 7, 14])
def test_what_is_not_finite_stays_in_its_row(N):
    lengths = np.random.default_rng(2).integers(0, 200, 3000)
    rng = np.random.default_rng(3)
    rowptr, colidx = wl.csr_from_lengths(rng, lengths, 5000)
    vals, B = wl.fill_values(rng, colidx.size, True), wl.fill_values(rng, 5000 * N, True).reshape(5000, N)
    vals[vals == 0] = 1
    B[7], B[4000] = np.inf, np.nan
    p = wl.SpmmProblem("narrow", 3000, 5000, N, rowptr, colidx, vals, B)
    got = DeviceProblem(p).run_cfg(binding.make_config(8, "parallel", "nnz_balanced")).cpu().numpy()
    with_7 = np.add.reduceat(np.append(colidx == 7, False), rowptr[:-1]).astype(bool) & (lengths > 0)
    with_4000 = np.add.reduceat(np.append(colidx == 4000, False), rowptr[:-1]).astype(bool) & (lengths > 0)
    assert np.isnan(got[with_4000]).all() and np.isinf(got[with_7 & ~with_4000]).all()
    assert np.isfinite(got[~with_7 & ~with_4000]).all()


@pytest.mark.parametrize("N", [1, 2, 3, 4, 7, 8, 13, 16])
def test_offsets_of_64_bits(N):
    """Columns on both sides of 4 GiB of B."""
    lengths = np.random.default_rng(N).integers(0, 60, 3000)
    rng, k = np.random.default_rng(3), 6200
    rowptr, colidx = wl.csr_from_lengths(rng, lengths, k)
    vals, B = wl.fill_values(rng, colidx.size, True), wl.fill_values(rng, k * N, True).reshape(k, N)
    ref, _ = oracle.spmm_csr(lengths.size, k, N, rowptr, colidx, vals, B, nthreads=8, bound=False)
    first = 2**32 // (4 * N) - k // 2
    wide = torch.zeros((first + k, N), device="cuda")
    wide[first:] = torch.from_numpy(B)
    C = torch.full((lengths.size, N), float("nan"), device="cuda")
    rp, ci, va = (torch.from_numpy(x).cuda() for x in (rowptr, colidx + np.int32(first), vals))
    binding.sgap_spmm_csr_cfg(lengths.size, first + k, N, rp, ci, va, wide, C, binding.make_config(8, "parallel", "nnz_balanced"))
    assert np.array_equal(C.cpu().numpy().astype(np.float64), ref)
