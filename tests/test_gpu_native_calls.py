"""The native call path of the binding: what it takes runs on the right stream, what it does not take is refused by the
binding's checks with the same errors as ever."""
import pytest
import torch

from paper_2209_02882_amd import binding
from paper_2209_02882_amd import workloads as wl

from gpu_util import DeviceProblem, assert_close, full_reference

pytestmark = pytest.mark.gpu


def test_streams_and_numbers_of_every_kind():
    import numpy as np

    p = wl.make_problem("uniform10_int")
    dp = DeviceProblem(p)
    ref, bnd = full_reference(p)
    args = (p.M, p.K, p.N, dp.rowptr, dp.colidx, dp.vals, dp.B)
    cfg = binding.make_config(8, "parallel", "row_split")
    side = torch.cuda.Stream()
    for how in ("current", "context", "explicit"):
        for call in (lambda C, s: binding.sgap_spmm_csr_ex(*args, C, 8, 0, 0, stream=s),
                     lambda C, s: binding.sgap_spmm_csr_ex(*args, C, np.int64(4), np.int32(1), 1, nnz_hint=-1, stream=s),
                     lambda C, s: binding.sgap_spmm_csr_cfg(*args, C, cfg, stream=s)):
            C = torch.full((p.M, p.N), float("nan"), device="cuda")
            torch.cuda.synchronize()
            if how == "context":
                with torch.cuda.stream(side):
                    torch.cuda._sleep(2_000_000)
                    call(C, None)
                    done = side.record_event()
                done.synchronize()  # of the side stream alone: the call has to be on it
            else:
                call(C, side if how == "explicit" else None)
                torch.cuda.synchronize()
            assert_close(C, ref, bnd, exact=True, what=how)


def test_what_is_wrong_is_still_said():
    p = wl.make_problem("uniform10_int")
    dp = DeviceProblem(p)
    C = dp.new_output()
    good = [p.M, p.K, p.N, dp.rowptr, dp.colidx, dp.vals, dp.B, C, 8, 0, 0]

    def broken(at, value):
        return good[:at] + [value] + good[at + 1:]

    for at, value, error in ((3, dp.rowptr[:-1], ValueError), (3, dp.rowptr.long(), TypeError), (4, dp.colidx.cpu(), TypeError),
                             (5, dp.vals.double(), TypeError), (6, dp.B.t(), ValueError), (7, C[:-1], ValueError),
                             (0, -1, Exception), (8, 3, binding.SgapError), (9, 7, binding.SgapError)):
        with pytest.raises(error):
            binding.sgap_spmm_csr_ex(*broken(at, value))
    with pytest.raises(TypeError):
        binding.sgap_spmm_csr_cfg(*good[:8], binding.make_config(8, "parallel", "row_split"), workspace=torch.zeros(4, device="cuda"))
