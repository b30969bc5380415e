"""SDDMM with four neighbouring rows together: rows, sharing and orders at which columns are listed or go one by one, long rows
dealt out by tiles, widths at the edges of lanes and of 64 columns; exact on integer-valued inputs."""
import functools

import numpy as np
import pytest
import torch

import oracle
from paper_2209_02882_amd import binding
from paper_2209_02882_amd import workloads as wl

from gpu_util import DeviceProblem

pytestmark = pytest.mark.gpu
ROWS, MORE_ROWS = 90_003, 170_003  # no multiples of four; a width of 128 wants more entries


def rows_of(kind):
    band = lambda r, n: r + np.arange(n)  # noqa: E731
    if kind == "band":
        return lambda r: band(r, 20)
    if kind == "30, 31 and 32 entries":  # few of 32: not more than a matrix has that goes by quads
        return lambda r: band(r, 32 if r in (1, 78, 207, 304, 396) else 30 + r // 8 % 2)
    if kind == "31 to 33 entries, entry by entry":
        return lambda r: band(r, 31 + r // 8 % 3 if r % 3 else 29)
    if kind == "in the row before the last":  # columns that come and go
        return lambda r: np.concatenate([band(r, 16), 600 + 30 * (r % 2) + np.arange(4)])
    if kind == "descending and repeated":
        return lambda r: band(r, 20)[::-1] if r % 40 == 3 else np.sort(np.concatenate([band(r, 16), band(r, 3)])) if r % 40 == 18 else band(r, 18)
    if kind == "with empty rows":
        return lambda r: band(r, 28) if r % 40 > 4 else band(0, 0)
    if kind == "nothing in common in places":
        return lambda r: band(r, 20) if r % 40 > 8 else 37 * (r % 8) + 41 * np.arange(17)
    long = {0: 255, 5: 256, 6: 511, 120: 7, 240: 513, 243: 40, 244: 3_000}  # of a period; the tiles have 256 or 512 entries
    return lambda r: band(r, long.get(r, 17))


KINDS = ["band", "30, 31 and 32 entries", "in the row before the last", "descending and repeated", "with empty rows",
         "nothing in common in places", "long rows", "31 to 33 entries, entry by entry"]


@functools.lru_cache
def csr(kind, rows=ROWS):
    """The rows of that kind, repeated with a period of 400 rows and shifted along."""
    period = [rows_of(kind)(r) for r in range(400)]
    columns = [period[r % 400] + 40 * (r // 400) for r in range(rows)]
    if kind == "long rows":  # in every other period: not more than a matrix has that goes by quads
        columns = [c if r // 400 % 2 else c[0] + np.arange(17) for r, c in enumerate(columns)]
        columns[-1] = np.arange(9_000)
    rowptr = np.concatenate([[0], np.cumsum([c.size for c in columns])]).astype(np.int32)
    assert (3_000_000 if rows == MORE_ROWS else 1_500_000) <= rowptr[-1] and 12 * rows < rowptr[-1] < 32 * rows
    return rowptr, np.concatenate(columns).astype(np.int32)


def problem(kind, J, rowptr, colidx):
    rng, K, rows = np.random.default_rng(J), int(colidx.max()) + 1, rowptr.size - 1
    p = wl.SpmmProblem(kind, rows, K, J, rowptr, colidx, wl.fill_values(rng, colidx.size, True),
                       wl.fill_values(rng, K * J, True).reshape(K, J))
    return p, wl.fill_values(rng, rows * J, True).reshape(rows, J)


def by_quads(p, g):
    return binding.load().sgap_debug_sddmm_quads(p.M, p.K, p.N, g, p.colidx.size, p.rowptr.ctypes.data, p.colidx.ctypes.data)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("J", [65, 68, 73, 101, 128, 129, 132, 137, 197, 256])
def test_rows_at_the_edges(J, kind):
    p, X1 = problem(kind, J, *csr(kind, MORE_ROWS if J == 128 else ROWS))
    ref, _ = oracle.sddmm_csr(p.M, p.K, p.N, p.rowptr, p.colidx, p.vals, X1, p.B)
    dp, X1d = DeviceProblem(p), torch.from_numpy(X1).cuda()
    for g in (8, 16, 32) if J <= 128 else (16, 32, 64):
        assert by_quads(p, g) == (kind != "31 to 33 entries, entry by entry" and J not in (65, 129) and (J, g) not in ((68, 32), (132, 64)))
        assert np.array_equal(dp.run_sddmm(X1d, g, "parallel").cpu().numpy().astype(np.float64), ref), g


def test_what_is_not_finite_stays_in_its_entries():
    J = 100
    p, X1 = problem("band", J, *csr("band"))
    p.vals[p.vals == 0] = 1
    p.B[70, 5], X1[300, 99] = np.inf, np.nan
    X1[:, 5] = 1
    assert by_quads(p, 8) == 1
    got = DeviceProblem(p).run_sddmm(torch.from_numpy(X1).cuda(), 8, "parallel").cpu().numpy()
    row = np.repeat(np.arange(ROWS), np.diff(p.rowptr))
    assert np.isnan(got[row == 300]).all()
    assert np.isinf(got[(p.colidx == 70) & (row != 300)]).all()
    assert np.isfinite(got[(p.colidx != 70) & (row != 300)]).all()


def test_small_products_are_kept():
    """Products and sums below the smallest normal number, as the fused multiply-adds have them."""
    J = 70
    p, X1 = problem("band", J, *csr("band"))
    p.vals[:] = 1
    p.B[:] = 0
    p.B[:, 7] = 2.0 ** -100
    X1[:] = 0
    X1[:, 7] = 2.0 ** -40
    assert by_quads(p, 8) == 1
    got = DeviceProblem(p).run_sddmm(torch.from_numpy(X1).cuda(), 8, "parallel").cpu().numpy()
    assert (got == np.float32(2.0 ** -140)).all()


@pytest.mark.parametrize("J", [68, 72, 75, 100, 128, 132, 136, 200, 256])
def test_no_less_exact_than_entry_by_entry(J):
    """Relative error (2-norm) against 64 bits, by quads and where the count of entries that is passed lets nothing look for them.
    Over a million entries and more the ratio of two such errors of alike sums is one within a few thousandths."""
    rowptr, colidx = csr("band", MORE_ROWS if J == 128 else ROWS)
    rows, K = rowptr.size - 1, int(colidx.max()) + 1
    rng = np.random.default_rng(J)
    p = wl.SpmmProblem("band", rows, K, J, rowptr, colidx, wl.fill_values(rng, colidx.size, False),
                       wl.fill_values(rng, K * J, False).reshape(K, J))
    X1 = wl.fill_values(rng, rows * J, False).reshape(rows, J)
    ref, _ = oracle.sddmm_csr(p.M, p.K, p.N, p.rowptr, p.colidx, p.vals, X1, p.B, nthreads=8, bound=False)
    dp, X1d = DeviceProblem(p), torch.from_numpy(X1).cuda()
    for g in [g for g in ((8, 16, 32) if J <= 128 else (16, 32, 64)) if (J, g) not in ((68, 32), (132, 64))]:
        assert by_quads(p, g) == 1
        error = []
        for hint in (colidx.size, 1):
            out = torch.full((colidx.size,), float("nan"), device="cuda")
            dp.launch_sddmm(X1d, out, g, "parallel", nnz_hint=hint)
            error.append(np.linalg.norm(out.cpu().numpy() - ref) / np.linalg.norm(ref))
        print(f"J={J} G={g} by quads {error[0]:.4g}, entry by entry {error[1]:.4g}", flush=True)
        assert error[0] <= 1.01 * error[1], g


@pytest.mark.parametrize("J", [100, 128, 250, 256])
def test_planes_dealt_over_the_dies(J):
    """Each die takes its share of every plane; the last planes are left over."""
    nx, ny, nz = 61, 103, 23
    at = np.arange(nx * ny * nz)
    x, y, z = at % nx, at // nx % ny, at // (nx * ny)
    columns, inside = [], []
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                inside.append((x + dx >= 0) & (x + dx < nx) & (y + dy >= 0) & (y + dy < ny) & (z + dz >= 0) & (z + dz < nz))
                columns.append((at + dx + nx * (dy + ny * dz)).astype(np.int32))
    inside, columns = np.stack(inside, 1), np.stack(columns, 1)
    p, X1 = problem("planes", J, np.concatenate([[0], np.cumsum(inside.sum(1))]).astype(np.int32), columns[inside])
    assert 3 * nx * ny * J * 4 > 4 << 20 and by_quads(p, 16) == 1
    ref, _ = oracle.sddmm_csr(p.M, p.K, p.N, p.rowptr, p.colidx, p.vals, X1, p.B, nthreads=8, bound=False)
    got = DeviceProblem(p).run_sddmm(torch.from_numpy(X1).cuda(), 16, "parallel").cpu().numpy()
    assert np.array_equal(got.astype(np.float64), ref)
