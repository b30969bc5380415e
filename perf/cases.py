"""The work that users of this library have it do, as cases that can be timed.

`listed()` names twelve of them; `draw(rng)` gives further ones of the same ranges.  The matrices and tensors follow
the recipes of paper_2209_02882_amd/workloads.py (uniform, power-law, 27-point stencil, R-MAT, skewed rows, compressed
sparse fibers), drawn on the GPU from the seed because they are made many times.  Every call goes through the binding
as an application's would, at a point of the design space that the library's own tuner or its defaults choose for that
kind of matrix.

Not here: the tuners and sgap_validate_csr (blocking calls, made once per matrix while a program is set up) and
sgap_reorder_rows_csr (a preparation too, and one with many correct results).
"""
from __future__ import annotations

import math

import torch

from paper_2209_02882_amd import binding

POWERLAW_EXPONENT, POWERLAW_SHIFT, POWERLAW_LONGEST = 2.1, 2.84, 4096  # mean row length 16
RMAT_A, RMAT_B, RMAT_C, RMAT_D = 0.57, 0.19, 0.19, 0.05
HEAVY_ROWS = 0.01  # skewed rows: this share of them is long
HEAVY_SLICES, HEAVY_FEWEST, HEAVY_MOST = 0.001, 2_000, 20_000  # skewed tensor: this share of its slices, their fibers
FIBER_LONGEST = 16
LONG_ROW_MIN = 1024


# --------------------------------------------------------------------------
# cases
# --------------------------------------------------------------------------

def _matrix(op, pattern, rows, columns, degree, n, group, strategy, schedule, windows=False):
    """`degree`: entries of a row, in the mean for a power law; of the longest row where rows are skewed."""
    return {"op": op, "pattern": pattern, "rows": rows, "columns": columns, "degree": degree, "n": n, "group": group,
            "strategy": strategy, "schedule": schedule, "windows": windows}


def _stencil(op, nx, ny, nz, n, group, strategy, schedule):
    return {"op": op, "pattern": "stencil27", "nx": nx, "ny": ny, "nz": nz, "n": n, "group": group, "strategy": strategy,
            "schedule": schedule, "windows": False}


def _rmat(op, scale, edges, n, group, strategy, schedule):
    return {"op": op, "pattern": "rmat", "scale": scale, "edges": edges, "n": n, "group": group, "strategy": strategy,
            "schedule": schedule, "windows": False}


def _tensor(op, slices, extent, fibers, skewed, n, group, strategy, schedule):
    return {"op": op, "pattern": "tensor", "slices": slices, "extent": extent, "fibers": fibers, "skewed": skewed, "n": n,
            "group": group, "strategy": strategy, "schedule": schedule}


def listed():
    named = {
        # one layer of a small graph, or one coarse level of a solver: the call is over in microseconds, and what it
        # costs is the way to the GPU; the library's default point
        "spmm_uniform_1k": _matrix("spmm", "uniform", 1024, 1024, 10, 32, 8, "parallel", "row_split"),
        # an ordinary graph with a few long rows, the tuner's choice for it
        "spmm_powerlaw_64k": _matrix("spmm", "powerlaw", 65_536, 65_536, 16, 64, 16, "serial", "nnz_balanced"),
        # the same kind at sizes that nothing divides: one column per lane, ragged last tiles, a matrix that is not square
        "spmm_powerlaw_ragged": _matrix("spmm", "powerlaw", 50_021, 61_657, 16, 37, 16, "parallel", "row_split"),
        # a discretised operator applied to a block of vectors
        "spmm_stencil_1m": _stencil("spmm", 100, 100, 100, 128, 1, "serial", "row_split"),
        # a large graph, node features of ordinary width
        "spmm_rmat_2m": _rmat("spmm", 21, 52_300_000, 32, 32, "serial", "nnz_balanced"),
        # the same graph with a few columns, the segmented reduction
        "spmm_rmat_2m_n4": _rmat("spmm", 21, 52_300_000, 4, 16, "parallel", "nnz_balanced"),
        # the largest: one row in a hundred holds nearly every entry, wide features, long rows by column windows
        "spmm_skewed_500k": _matrix("spmm", "skewed", 500_000, 500_000, 20_000, 256, 2, "serial", "row_split", True),
        # the sampled product on a pattern: the gradient of SpMM with respect to the values of A, attention scores
        "sddmm_stencil_1m": _stencil("sddmm", 100, 100, 100, 128, 8, "parallel", "nnz_balanced"),
        "sddmm_skewed_500k": _matrix("sddmm", "skewed", 500_000, 500_000, 20_000, 256, 8, "parallel", "nnz_balanced", True),
        # tensor decompositions: slices that are alike, slices of which a few are huge, and one mode product
        "mttkrp_tensor_262k": _tensor("mttkrp", 262_144, 65_536, 8, False, 32, 8, "parallel", "row_split"),
        "mttkrp_skewed_262k": _tensor("mttkrp", 262_144, 65_536, 4, True, 32, 32, "serial", "nnz_balanced"),
        "ttm_tensor_262k": _tensor("ttm", 262_144, 65_536, 8, False, 32, 2, "serial", "row_split"),
    }
    return [dict(case, name=name) for name, case in named.items()]


def _between(rng, lo, hi):
    """A whole number of [lo, hi], spread over the logarithm."""
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def _of_four(n):
    return n // 4 * 4


def draw(rng):
    """One case of the ranges that the listed ones stand for."""
    kind = rng.choice(("uniform", "powerlaw", "powerlaw_rows", "stencil", "rmat", "rmat_narrow", "skewed", "sddmm",
                       "sddmm_skewed", "mttkrp", "mttkrp_skewed", "ttm"))
    if kind == "uniform":
        point = rng.choice(((8, "parallel", "row_split"), (4, "parallel", "row_split"), (1, "serial", "row_split"),
                            (8, "serial", "nnz_balanced")))
        return _matrix("spmm", "uniform", _between(rng, 500, 60_000), _between(rng, 500, 60_000), rng.randint(4, 32),
                       _between(rng, 1, 64), *point)
    if kind == "powerlaw":
        point = rng.choice(((8, "serial", "nnz_balanced"), (16, "serial", "nnz_balanced"), (32, "serial", "nnz_balanced")))
        return _matrix("spmm", "powerlaw", _between(rng, 8_000, 300_000), _between(rng, 8_000, 300_000), 16,
                       _between(rng, 16, 128), *point)
    if kind == "powerlaw_rows":
        point = rng.choice(((8, "parallel", "row_split"), (16, "parallel", "row_split"), (32, "parallel", "row_split")))
        return _matrix("spmm", "powerlaw", _between(rng, 8_000, 200_000), _between(rng, 8_000, 200_000), 16,
                       _between(rng, 4, 64), *point)
    if kind in ("stencil", "sddmm") and (kind == "stencil" or rng.random() < 0.5):
        box = [rng.randint(30, 100) for _ in range(3)]
        if kind == "sddmm":
            return _stencil("sddmm", *box, _between(rng, 32, 128), rng.choice((8, 16)), "parallel", "nnz_balanced")
        return _stencil("spmm", *box, _between(rng, 16, 128), rng.choice((1, 2)), "serial", "row_split")
    if kind in ("rmat", "rmat_narrow", "sddmm"):
        scale = rng.randint(15, 21)
        edges = int((1 << scale) * rng.uniform(8, 25))
        if kind == "sddmm":
            return _rmat("sddmm", scale, edges, _between(rng, 16, 64), rng.choice((4, 8)), "parallel", "nnz_balanced")
        if kind == "rmat":
            return _rmat("spmm", scale, edges, _between(rng, 16, 64), rng.choice((16, 32, 64)), "serial", "nnz_balanced")
        return _rmat("spmm", scale, edges, rng.choice((1, 2, 4, 8)), rng.choice((8, 16)), "parallel", "nnz_balanced")
    if kind in ("skewed", "sddmm_skewed"):
        rows = _between(rng, 60_000, 500_000)
        longest = min(20_000, rows // 8)
        if kind == "skewed":
            return _matrix("spmm", "skewed", rows, rows, longest, _of_four(rng.randint(64, 256)), rng.choice((1, 2, 4)),
                           "serial", "row_split", True)
        return _matrix("sddmm", "skewed", rows, rows, longest, _of_four(rng.randint(64, 256)), 8, "parallel",
                       "nnz_balanced", True)
    slices, extent = _between(rng, 10_000, 262_144), _between(rng, 20_000, 65_536)
    n = rng.choice((16, 24, 32, 48, 64))
    if kind == "mttkrp":
        return _tensor("mttkrp", slices, extent, rng.randint(4, 8), False, min(n, 32), rng.choice((4, 8)), "parallel", "row_split")
    if kind == "mttkrp_skewed":
        return _tensor("mttkrp", slices, extent, 4, True, min(n, 32), rng.choice((16, 32)), "serial", "nnz_balanced")
    return _tensor("ttm", slices, extent, rng.randint(4, 8), False, n, rng.choice((1, 2, 4)), "serial", "row_split")


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------

def _values(gen, *shape):
    """Uniform on [-1, 1)."""
    return torch.rand(shape, generator=gen, device="cuda").mul_(2).sub_(1)


def _distinct(gen, keys, rows, columns, entries=None):
    """CSR structure of the distinct (row * columns + column) keys; of `entries` of them, where the number has to be
    the same for every seed because a result has one element or one row for each."""
    keys = torch.unique(keys)
    if entries is not None:
        keep = torch.ones_like(keys, dtype=torch.bool)
        keep[torch.randperm(keys.numel(), generator=gen, device="cuda")[:keys.numel() - entries]] = False
        keys = keys[keep]
    rowptr = torch.searchsorted(keys, torch.arange(rows + 1, device="cuda") * columns).to(torch.int32)
    return rowptr, (keys % columns).to(torch.int32)


def _rows_of(gen, lengths, columns, entries=None):
    """Rows of the given lengths, columns uniform, repeated draws dropped, sorted inside a row."""
    rows = torch.repeat_interleave(torch.arange(lengths.numel(), device="cuda"), lengths)
    keys = rows * columns + torch.randint(columns, rows.shape, generator=gen, device="cuda")
    return _distinct(gen, keys, lengths.numel(), columns, entries)


def _stencil_rows(nx, ny, nz):
    """27-point stencil on a box in natural order, clipped at the faces."""
    at = torch.arange(nx * ny * nz, device="cuda")
    x, y, z = at % nx, at // nx % ny, at // (nx * ny)
    columns, inside = [], []
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                inside.append((x + dx >= 0) & (x + dx < nx) & (y + dy >= 0) & (y + dy < ny) & (z + dz >= 0) & (z + dz < nz))
                columns.append((at + dx + nx * (dy + ny * dz)).to(torch.int32))
    inside, columns = torch.stack(inside, 1), torch.stack(columns, 1)
    rowptr = torch.zeros(at.numel() + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = torch.cumsum(inside.sum(1), 0)
    return rowptr, columns[inside]


def _rmat_rows(gen, scale, edges, entries):
    row = torch.zeros(edges, dtype=torch.int64, device="cuda")
    column = torch.zeros_like(row)
    for _ in range(scale):
        u = torch.rand(edges, generator=gen, device="cuda")
        down = u >= RMAT_A + RMAT_B
        right = ((u >= RMAT_A) & ~down) | (u >= RMAT_A + RMAT_B + RMAT_C)
        row = row * 2 + down
        column = column * 2 + right
    return _distinct(gen, row * (1 << scale) + column, 1 << scale, 1 << scale, entries)


def _skewed_lengths(m, longest, device="cuda"):
    """Lengths spread evenly over [longest / 10, longest] for the long rows and over 1 to 8 for the others."""
    heavy = round(m * HEAVY_ROWS)
    return torch.cat([torch.linspace(longest / 10, longest, heavy, device=device).long(), torch.arange(m - heavy, device=device) % 8 + 1])


def _csr(case, gen):
    """(rows, columns, rowptr, colidx) of a matrix case."""
    m, k, entries = _entries(case)
    entries = int(entries - 6 * math.sqrt(entries)) if case["op"] == "sddmm" else None
    if case["pattern"] == "stencil27":
        return (m, k, *_stencil_rows(case["nx"], case["ny"], case["nz"]))
    if case["pattern"] == "rmat":
        return (m, k, *_rmat_rows(gen, case["scale"], case["edges"], entries))
    if case["pattern"] == "uniform":
        lengths = torch.full((m,), case["degree"], device="cuda")
    elif case["pattern"] == "powerlaw":
        weights = (torch.arange(1, POWERLAW_LONGEST + 1, device="cuda", dtype=torch.float64) + POWERLAW_SHIFT) ** -POWERLAW_EXPONENT
        share = torch.cumsum(weights / weights.sum(), 0)
        lengths = 1 + torch.searchsorted(share, torch.rand(m, generator=gen, device="cuda", dtype=torch.float64), right=True)
        lengths.clamp_(max=POWERLAW_LONGEST)
    else:
        lengths = _skewed_lengths(m, case["degree"])[torch.randperm(m, generator=gen, device="cuda")]
    return (m, k, *_rows_of(gen, lengths, k, entries))


def _packed(operands, *shape):
    """The operands and a result of that shape in one allocation, one after the other at 512-byte boundaries: the
    placement that include/sgap.h recommends for operands that are multiplied many times."""
    sizes = [t.numel() * 4 for t in operands] + [4 * math.prod(shape)]
    starts, end = [], 0
    for size in sizes:
        starts.append(end)
        end += -(-size // 512) * 512
    arena = torch.zeros(end, dtype=torch.uint8, device="cuda")
    placed = []
    for t, start, size in zip(operands, starts, sizes):
        placed.append(arena[start:start + size].view(t.dtype).view(t.shape))
        placed[-1].copy_(t)
    return placed, arena[starts[-1]:starts[-1] + sizes[-1]].view(torch.float32).view(shape)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    group, n = case["group"], case["n"]
    strategy, schedule = binding.STRATEGIES[case["strategy"]], binding.SCHEDULES[case["schedule"]]
    if case["pattern"] == "tensor":
        slices, extent = case["slices"], case["extent"]
        lengths = torch.empty(slices, dtype=torch.int64, device="cuda").geometric_(1 / case["fibers"], generator=gen)
        lengths -= (torch.rand(slices, generator=gen, device="cuda") < 0.125).long()
        if case["skewed"]:
            heavy = torch.randperm(slices, generator=gen, device="cuda")[:round(slices * HEAVY_SLICES)]
            lengths[heavy] = torch.randint(HEAVY_FEWEST, HEAVY_MOST + 1, heavy.shape, generator=gen, device="cuda")
        fptr, fidx = _rows_of(gen, lengths, extent, int(_fibers(case) - 6 * case["fibers"] * math.sqrt(slices)) if case["op"] == "ttm" else None)
        eptr, eidx = _rows_of(gen, torch.randint(1, FIBER_LONGEST + 1, fidx.shape, generator=gen, device="cuda"), extent)
        vals, left, right = _values(gen, eidx.numel()), _values(gen, extent, n), _values(gen, extent, n)
        if case["op"] == "ttm":
            (eptr, eidx, vals, right), out = _packed((eptr, eidx, vals, right), fidx.numel(), n)
            return binding.sgap_ttm_csf, (fidx.numel(), extent, n, eptr, eidx, vals, right, out, group, strategy, schedule), {}, out
        (fptr, fidx, eptr, eidx, vals, left, right), out = _packed((fptr, fidx, eptr, eidx, vals, left, right), slices, n)
        return binding.sgap_mttkrp_csf_ex, (slices, extent, extent, n, fptr, fidx, eptr, eidx, vals, left, right, out,
                                            group, strategy, schedule), {}, out
    m, k, rowptr, colidx = _csr(case, gen)
    vals, dense = _values(gen, colidx.numel()), _values(gen, k, n)
    if case["op"] == "sddmm":
        (rowptr, colidx, vals, left, dense), out = _packed((rowptr, colidx, vals, _values(gen, m, n), dense), colidx.numel())
        operands = (m, k, n, rowptr, colidx, vals, left, dense, out, group, strategy)
        if not case["windows"]:
            return binding.sgap_sddmm_csr, operands, {}, out
        workspace = torch.empty(binding.sgap_sddmm_csr_workspace_size(k, n), dtype=torch.uint8, device="cuda")
        return binding.sgap_sddmm_csr_windows, (*operands, LONG_ROW_MIN), {"workspace": workspace}, out
    (rowptr, colidx, vals, dense), out = _packed((rowptr, colidx, vals, dense), m, n)
    operands = (m, k, n, rowptr, colidx, vals, dense, out)
    if not case["windows"]:
        return binding.sgap_spmm_csr_ex, (*operands, group, strategy, schedule), {}, out
    config = binding.make_config(group, strategy, schedule, long_row_min=LONG_ROW_MIN)
    workspace = torch.empty(binding.sgap_spmm_csr_workspace_size(m, k, n, config), dtype=torch.uint8, device="cuda")
    return binding.sgap_spmm_csr_cfg, (*operands, config), {"workspace": workspace}, out


def run(state):
    call, operands, options, out = state
    call(*operands, **options)
    return out


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------

def _entries(case):
    """(rows, columns, expected stored entries) of a matrix case."""
    if case["pattern"] == "stencil27":
        m = case["nx"] * case["ny"] * case["nz"]
        return m, m, math.prod(3 * case[d] - 2 for d in ("nx", "ny", "nz"))
    if case["pattern"] == "rmat":
        # distinct cells among `edges` throws: a cell of i, j, k, l levels in each quadrant is hit with probability
        # a^i b^j c^k d^l; b == c, so the two are counted together
        scale, edges, total = case["scale"], case["edges"], 0.0
        for i in range(scale + 1):
            for j in range(scale + 1 - i):
                l = scale - i - j
                cells = math.comb(scale, i) * math.comb(scale - i, j) * 2.0 ** j
                p = RMAT_A ** i * RMAT_B ** j * RMAT_D ** l
                total += cells * -math.expm1(edges * math.log1p(-p))
        return 1 << scale, 1 << scale, total
    m, k = case["rows"], case["columns"]
    if case["pattern"] == "skewed":
        lengths = _skewed_lengths(m, case["degree"], "cpu").double()
        return m, k, float((-k * torch.expm1(-lengths / k)).sum())
    return m, k, m * case["degree"]


def _fibers(case):
    """Expected stored fibers of a tensor case."""
    fibers = case["slices"] * (case["fibers"] - 0.125)
    if case["skewed"]:
        fibers = fibers * (1 - HEAVY_SLICES) + case["slices"] * HEAVY_SLICES * (HEAVY_FEWEST + HEAVY_MOST) / 2
    return fibers


def work(case):
    n = case["n"]
    if case["pattern"] == "tensor":
        slices, extent = case["slices"], case["extent"]
        fibers = _fibers(case)
        entries = fibers * (1 + FIBER_LONGEST) / 2
        if case["op"] == "ttm":
            return {"bytes": entries * 8 + fibers * 4 + (extent + fibers) * n * 4, "flops": 2 * entries * n}
        return {"bytes": entries * 8 + fibers * 8 + slices * 4 + (2 * extent + slices) * n * 4, "flops": 2 * n * (entries + fibers)}
    m, k, entries = _entries(case)
    per_entry = 12 if case["op"] == "sddmm" else 8  # column and value in, for the sampled product one value out
    return {"bytes": entries * per_entry + (m + 1) * 4 + (k + m) * n * 4, "flops": 2 * entries * n}


def tolerance(case):
    """fp32 operands, products and sums; the order of the additions is the implementation's."""
    return {"rel": 1e-5}
