"""The binding where its native module has not been built: the calls work through ctypes."""
import sys

import pytest
import torch

import paper_2209_02882_amd
from paper_2209_02882_amd import binding
from paper_2209_02882_amd import workloads as wl


@pytest.fixture
def without_native(monkeypatch):
    monkeypatch.setitem(sys.modules, "paper_2209_02882_amd._native", None)
    monkeypatch.delattr(paper_2209_02882_amd, "_native", raising=False)
    monkeypatch.setattr(binding, "_native", None)


def test_the_checks_are_reached_and_a_warning_is_given(without_native):
    ints, floats = torch.zeros(2, dtype=torch.int32), torch.zeros(1)
    with pytest.warns(RuntimeWarning, match="ctypes"), pytest.raises(TypeError, match="CUDA tensor"):
        binding.sgap_spmm_csr_ex(1, 1, 1, ints, ints[:1], floats, floats, floats, 8, 0, 0)
    with pytest.raises(TypeError, match="CUDA tensor"):
        binding.sgap_sddmm_csr(1, 1, 1, ints, ints[:1], floats, floats, floats, floats, 8, 0)


@pytest.mark.gpu
def test_every_call_works(without_native):
    import oracle
    from gpu_util import DeviceProblem, assert_close, full_reference
    from paper_2209_02882_amd.device import DeviceTensor3

    p = wl.make_problem("uniform10_int")
    dp = DeviceProblem(p)
    ref, bnd = full_reference(p)
    with pytest.warns(RuntimeWarning, match="ctypes"):
        assert_close(dp.run(8, "parallel", "row_split"), ref, bnd, exact=True)
    config = binding.make_config(2, "serial", "row_split", long_row_min=8)
    assert_close(dp.run_cfg(config), ref, bnd, exact=True)
    X1 = wl.sddmm_left_operand(p)
    ref, bnd = oracle.sddmm_csr(p.M, p.K, p.N, p.rowptr, p.colidx, p.vals, X1, p.B)
    for out in (dp.run_sddmm(torch.from_numpy(X1).cuda(), 8, "parallel"),
                dp.run_sddmm_windows(torch.from_numpy(X1).cuda(), 8, "parallel", 8)):
        assert (abs(out.cpu().numpy() - ref) <= 1e-5 * bnd).all()
    t = wl.make_tensor3("tensor3_small_int")
    dt = DeviceTensor3(t)
    ref, bnd = oracle.mttkrp_csf(t.I, t.K, t.L, t.J, t.fptr, t.fidx, t.eptr, t.eidx, t.vals, t.X1, t.X2)
    assert_close(dt.run_mttkrp(8, "parallel", "nnz_balanced"), ref, bnd, exact=True)
    ref, bnd = oracle.ttm_csf(t.I, t.K, t.L, t.J, t.fptr, t.fidx, t.eptr, t.eidx, t.vals, t.X2)
    assert_close(dt.run_ttm(2, "serial", "row_split"), ref, bnd, exact=True)
