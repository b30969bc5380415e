"""Row-split, serial strategy, four neighbouring rows together: rows, sharing and orders at which a quad is listed or goes row by
row, widths at the edges of lanes and column tiles, planes dealt over the dies; exact on integer-valued inputs."""
import ctypes
import functools

import numpy as np
import pytest
import torch

import oracle
from paper_2209_02882_amd import binding
from paper_2209_02882_amd import workloads as wl

from gpu_util import DeviceProblem

pytestmark = pytest.mark.gpu
ROWS, MORE_ROWS = 82_003, 150_003  # no multiples of four; up to 64 columns want more blocks of them (check asserts that they are enough)


@functools.lru_cache
def csr(kind, N=128):
    """The rows of that kind, repeated with a period of 400 rows and shifted along."""
    period = [rows_of(kind)(r) for r in range(400)]
    columns = [period[r % 400] + 40 * (r // 400) for r in range(MORE_ROWS if N <= 64 else ROWS)]
    rowptr = np.concatenate([[0], np.cumsum([c.size for c in columns])]).astype(np.int32)
    return rowptr, np.concatenate(columns).astype(np.int32)


def rows_of(kind):
    rng = np.random.default_rng(7)
    band = lambda r, n: r + np.arange(n)  # noqa: E731
    some = [np.sort(rng.choice(900, n, replace=False)) for n in rng.integers(0, 41, 400)]
    if kind == "band":
        return lambda r: band(r, 20)
    if kind == "31, 32 and 33 entries":
        return lambda r: band(r, 31 + r // 8 % 3)
    if kind == "as many records as there is room for, and one more":
        return lambda r: np.sort(np.concatenate([np.arange(20 - r // 4 % 3), 900 + 11 * (r % 4) + np.arange(11 + r // 4 % 3)]))
    if kind == "in the row before the last":  # columns that come and go
        return lambda r: np.concatenate([band(r, 14), 600 + 30 * (r % 2) + np.arange(6)])
    if kind == "descending and repeated":
        return lambda r: band(r, 20)[::-1] if r % 8 < 4 and r % 3 == 0 else np.sort(np.concatenate([band(r, 16), band(r, 3)])) if r % 16 > 12 else band(r, 18)
    if kind == "no column in common within the first two, or the last two":
        return lambda r: np.concatenate([band(r, 18) + 500 * (r % 4 > (0, 2)[r // 4 % 2])])
    if kind == "long rows":  # quads of 160 entries and one more, and of more than are read at a time; a wavefront's quads among them
        long = {0: 100, 4: 101, 9: 79, 10: 80, 11: 81, 14: 160, 40: 161, 41: 0, 42: 0, 43: 0, 200: 41, 204: 700, 205: 321, 206: 33, 399: 160}
        return lambda r: band(r, long.get(r, 20))
    if kind == "with empty rows":
        return lambda r: band(r, 28 if r % 5 else 0) if r % 40 > 3 else band(0, 0)
    return lambda r: some[r]  # without order


KINDS = ["band", "31, 32 and 33 entries", "as many records as there is room for, and one more", "in the row before the last",
         "descending and repeated",
         "no column in common within the first two, or the last two", "with empty rows", "without order", "long rows"]


def check(p, points, quads=1, **knobs):
    units = torch.cuda.get_device_properties(0).multi_processor_count
    ref, _ = oracle.spmm_csr(p.M, p.K, p.N, p.rowptr, p.colidx, p.vals, p.B, nthreads=8, bound=False)
    dp = DeviceProblem(p)
    for g in points:
        cfg = binding.make_config(g, "serial", "row_split", **knobs)
        assert binding.load().sgap_debug_row_quads(p.M, p.N, p.colidx.size, ctypes.byref(cfg), units) == quads
        assert np.array_equal(dp.run_cfg(cfg).cpu().numpy().astype(np.float64), ref), (g, knobs)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("N", [61, 64, 66, 130, 260])
def test_rows_at_the_edges(N, kind):
    rowptr, colidx = csr(kind, N)
    rng, K = np.random.default_rng(N), int(colidx.max()) + 1
    p = wl.SpmmProblem("quads", rowptr.size - 1, K, N, rowptr, colidx, wl.fill_values(rng, colidx.size, True),
                       wl.fill_values(rng, K * N, True).reshape(K, N))
    check(p, (1, 4))
    if N == 260:
        check(p, (2,), tile_cols=256)  # 64 lanes to a row
    if kind == "band":
        check(p, (1,), xcd_remap=0)


@pytest.mark.parametrize("N,tile_cols", [(260, 260), (300, 300), (300, 1000), (520, 512), (520, 300), (600, 1000)])
def test_column_tiles_wider_than_a_wavefront(N, tile_cols):
    """64 lanes hold 256 columns: a tile of more takes several passes over its rows."""
    rowptr, colidx = csr("band")
    rng, K = np.random.default_rng(N), int(colidx.max()) + 1
    p = wl.SpmmProblem("quads", ROWS, K, N, rowptr, colidx, wl.fill_values(rng, colidx.size, True),
                       wl.fill_values(rng, K * N, True).reshape(K, N))
    check(p, (1, 2, 4), quads=0, tile_cols=tile_cols)


@pytest.mark.parametrize("N", [40, 64, 100, 132])  # 40: the rows as they are decide, not the lanes they take
def test_planes_dealt_over_the_dies(N):
    nx, ny, nz = 61, 103, 19 if N > 64 else 23  # reach 6,345 rows, the last planes are left over
    x, y, z = (v.ravel() for v in np.meshgrid(np.arange(nx), np.arange(ny), np.arange(nz), indexing="ij"))
    order = np.lexsort((x, y, z))
    x, y, z = x[order], y[order], z[order]
    columns, inside = [], []
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                inside.append((x + dx >= 0) & (x + dx < nx) & (y + dy >= 0) & (y + dy < ny) & (z + dz >= 0) & (z + dz < nz))
                columns.append(x + dx + nx * (y + dy + ny * (z + dz)))
    inside, columns = np.stack(inside, 1), np.stack(columns, 1)
    M = nx * ny * nz
    rowptr = np.concatenate([[0], np.cumsum(inside.sum(1))]).astype(np.int32)
    colidx = columns[inside].astype(np.int32)
    rng = np.random.default_rng(N)
    p = wl.SpmmProblem("planes", M, M, N, rowptr, colidx, wl.fill_values(rng, colidx.size, True),
                       wl.fill_values(rng, M * N, True).reshape(M, N))
    check(p, (1,))


@pytest.mark.parametrize("kind", ["band", "no column in common within the first two, or the last two", "31, 32 and 33 entries", "long rows"])
@pytest.mark.parametrize("N,tile_cols", [(61, 0), (64, 0), (128, 0), (256, 256)])  # 16, 32 and 64 lanes
def test_what_is_not_finite_stays_in_its_rows(N, tile_cols, kind):
    """Listed quads that are done again beside quads whose rows go one by one, from LDS and from memory."""
    rowptr, colidx = csr(kind, N)
    rng, K = np.random.default_rng(3), int(colidx.max()) + 1
    vals, B = wl.fill_values(rng, colidx.size, True), wl.fill_values(rng, K * N, True).reshape(K, N)
    vals[vals == 0] = 1
    ref, _ = oracle.spmm_csr(rowptr.size - 1, K, N, rowptr, colidx, vals, B, nthreads=8, bound=False)
    infinite = np.concatenate([[70], np.arange(3_000, K, 157)])
    B[infinite, 5], B[300, 60] = np.inf, np.nan
    p = wl.SpmmProblem("quads", rowptr.size - 1, K, N, rowptr, colidx, vals, B)
    cfg = binding.make_config(1, "serial", "row_split", tile_cols=tile_cols)
    units = torch.cuda.get_device_properties(0).multi_processor_count
    assert binding.load().sgap_debug_row_quads(p.M, N, colidx.size, ctypes.byref(cfg), units) == 1
    got = DeviceProblem(p).run_cfg(cfg).cpu().numpy()
    has = lambda c: (np.diff(rowptr) > 0) & (np.add.reduceat(np.append(np.isin(colidx, c), False), rowptr[:-1]) > 0)  # noqa: E731
    assert not np.isfinite(got[has(infinite), 5]).any() and np.isnan(got[has([300]), 60]).all()
    rest = np.ones(got.shape, bool)
    rest[has(infinite), 5] = rest[has([300]), 60] = False
    assert np.array_equal(got[rest].astype(np.float64), ref[rest])


@pytest.mark.parametrize("N,tile_cols", [(64, 0), (61, 0), (128, 0), (256, 256)])  # 16, 32 and 64 lanes
def test_offsets_of_64_bits(N, tile_cols):
    """Columns on both sides of 4 GiB of B."""
    rowptr, colidx = csr("long rows", N)
    rng, k = np.random.default_rng(N), int(colidx.max()) + 1
    vals, B = wl.fill_values(rng, colidx.size, True), wl.fill_values(rng, k * N, True).reshape(k, N)
    ref, _ = oracle.spmm_csr(rowptr.size - 1, k, N, rowptr, colidx, vals, B, nthreads=8, bound=False)
    first = 2**32 // (4 * N) - k // 2
    wide = torch.zeros((first + k, N), device="cuda")
    wide[first:] = torch.from_numpy(B)
    C = torch.full((rowptr.size - 1, N), float("nan"), device="cuda")
    rp, ci, va = (torch.from_numpy(x).cuda() for x in (rowptr, colidx + np.int32(first), vals))
    cfg = binding.make_config(1, "serial", "row_split", tile_cols=tile_cols)
    units = torch.cuda.get_device_properties(0).multi_processor_count
    assert binding.load().sgap_debug_row_quads(rowptr.size - 1, N, colidx.size, ctypes.byref(cfg), units) == 1
    binding.sgap_spmm_csr_cfg(rowptr.size - 1, first + k, N, rp, ci, va, wide, C, cfg)
    assert np.array_equal(C.cpu().numpy().astype(np.float64), ref)
