"""MTTKRP by blocks of slices (parallel strategy): pieces of a block, slices that go on in the next one, and fibers that a
piece has no room for (3,328 entries, 512 fibers).  Exact on integer values."""
import numpy as np
import pytest
import torch

import oracle
from paper_2209_02882_amd import binding
from paper_2209_02882_amd import workloads as wl

pytestmark = pytest.mark.gpu


def tensor(I, K, L, J, fibers, entries, seed):
    rng = np.random.default_rng(seed)
    fptr, fidx = wl.csr_from_lengths(rng, np.asarray(fibers, dtype=np.int64), K)
    eptr, eidx = wl.csr_from_lengths(rng, np.resize(np.asarray(entries, dtype=np.int64), int(fptr[-1])), L)
    vals = wl.fill_values(rng, int(eptr[-1]), True)
    return wl.Tensor3Problem("custom", I, K, L, J, fptr, fidx, eptr, eidx, vals, wl.fill_values(rng, K * J, True).reshape(K, J),
                             wl.fill_values(rng, L * J, True).reshape(L, J))


CASES = {
    # the room of a piece, one less and one more, alone and between others; fibers without entries at both ends
    "long_fibers": ([0, 1, 3, 0, 2, 5, 1, 1, 4], [0, 3327, 3328, 3329, 6656, 1, 6657, 0, 2, 9985, 0]),
    # a slice over many pieces, more than 512 fibers of an entry or none each, and short slices around it
    "many_fibers": ([1, 0, 2, 1700, 1, 0, 511, 512, 513, 3], [1, 0, 2]),
    # pieces that end with a slice, in the middle of one, and before a fiber that would not fit
    "full_pieces": ([7, 7, 7, 14, 1, 0, 20, 9], [512]),
    "single": ([1], [1]),
    # more slices without fibers than a piece of a tile keeps pointers of (256), in front, between and behind
    "empty_slices": ([0] * 300 + [3, 0, 2] + [0] * 700 + [900] + [0] * 255 + [1] + [0] * 256 + [5, 4] + [0] * 300, [9, 1, 0, 30]),
}


@pytest.mark.parametrize("J", [1, 2, 3, 4, 7, 32, 33, 100, 260])
@pytest.mark.parametrize("name", list(CASES))
def test_pieces_of_a_block(name, J):
    fibers, entries = CASES[name]
    t = tensor(len(fibers), 2000, 11000 if J < 100 else 10800, J, fibers, entries, seed=J)
    ref, _ = oracle.mttkrp_csf(t.I, t.K, t.L, t.J, t.fptr, t.fidx, t.eptr, t.eidx, t.vals, t.X1, t.X2, nthreads=8)
    d = [torch.from_numpy(x).cuda() for x in (t.fptr, t.fidx, t.eptr, t.eidx, t.vals, t.X1, t.X2)]
    Y = torch.empty((t.I, t.J), device="cuda")
    for hint in (-1, 0, 1, t.nnz, 10**9):  # 16 slices to a block, 256, and down to one
        for g in (1, 8):
            print("  mttkrp", name, J, hint, g, flush=True)
            Y.fill_(float("nan"))
            binding.sgap_mttkrp_csf_ex(t.I, t.K, t.L, t.J, *d, Y, g, binding.SGAP_REDUCE_PARALLEL, binding.SGAP_SCHED_ROW_SPLIT, nnz_hint=hint)
            assert np.array_equal(Y.cpu().numpy().astype(np.float64), ref), (hint, g)
        # the same pieces from tiles of stored entries, of 1,024 to 2,000 each (few of few columns: shares of lanes), slices merged where they reach beyond one
        print("  mttkrp tiles", name, J, hint, flush=True)
        Y.fill_(float("nan"))
        binding.sgap_mttkrp_csf_ex(t.I, t.K, t.L, t.J, *d, Y, 8, binding.SGAP_REDUCE_SERIAL, binding.SGAP_SCHED_NNZ_BALANCED, nnz_hint=hint)
        assert np.array_equal(Y.cpu().numpy().astype(np.float64), ref), hint
