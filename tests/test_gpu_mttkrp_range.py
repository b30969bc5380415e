"""MTTKRP multiplies an entry with its row of X2 first and the row of X1 last (the fiber's sum comes before the factor of
the fiber): values that meet in range in that order, and only in that order, give the exact result at every point."""
import numpy as np
import pytest

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
