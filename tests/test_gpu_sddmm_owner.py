"""SDDMM with long rows by column windows (windows of 64 KiB lie in LDS; of 160 KiB owner wavefronts take them, from 129 columns
on, in lists of 256 rows and more), the short rows' kernel beside them, and the rows that fall to neither: exact on
integer-valued inputs."""
import numpy as np
import pytest
import torch

import oracle
from paper_2209_02882_amd import workloads as wl

from gpu_util import DeviceProblem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("J", [32, 64, 100, 128, 132, 200, 252, 256])
@pytest.mark.parametrize("min_len,window_kb,cap", [(150, 0, 0), (150, 64, 0), (150, 160, 0), (1500, 256, 0), (40, 16, 255)])
def test_long_short_and_other_rows(J, min_len, window_kb, cap):
    rng = np.random.default_rng(J + min_len)
    M, K = 3000, 5000
    lengths = rng.integers(0, 20, M)
    long = rng.choice(M, 700, replace=False)
    lengths[long] = rng.integers(30, 400, 700)
    lengths[long[:40]] = rng.integers(900, 2500, 40)  # below and above the rows the short rows' kernel takes
    rowptr, colidx = wl.csr_from_lengths(rng, lengths, K)
    vals = wl.fill_values(rng, colidx.size, True)
    B = wl.fill_values(rng, K * J, True).reshape(K, J)
    X1 = wl.fill_values(rng, M * J, True).reshape(M, J)
    p = wl.SpmmProblem("owner", M, K, J, rowptr, colidx, vals, B)
    ref, _ = oracle.sddmm_csr(M, K, J, rowptr, colidx, vals, X1, B, nthreads=8, bound=False)
    dp = DeviceProblem(p)
    X1d = torch.from_numpy(X1).cuda()
    for g, st in ((8, "parallel"), (4, "serial")):
        got = dp.run_sddmm_windows(X1d, g, st, min_len, window_kb, cap).cpu().numpy().astype(np.float64)
        assert np.array_equal(got, ref), (g, st)
