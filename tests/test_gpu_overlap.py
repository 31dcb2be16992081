"""The choice of the overlapped reverse sweep: by what a context holds beside the
line kernels' copy of the factors, so that keeping the copy takes it from no
grid that had it."""
import pytest

import tc_inputs

pytestmark = pytest.mark.gpu


def test_line_copy_does_not_end_the_overlap(monkeypatch):
    import torch
    from paper_1311_2481_amd import Solver
    from paper_1311_2481_amd.autograd import TWIN_MAX_BYTES, TCSteps
    args = (16, 488, 976, 0.5, 100.0, 0.0, 1e-8)
    monkeypatch.setenv("TC_PC_LINE", "0")
    S = Solver(*args)
    without = S.memory_bytes()
    assert S.line_copy_bytes() == 0
    S.close()
    monkeypatch.delenv("TC_PC_LINE")
    S = Solver(*args)
    assert S.memory_bytes() - S.line_copy_bytes() == without
    assert without <= TWIN_MAX_BYTES < S.memory_bytes()
    x = S.zeros(3).requires_grad_(True)
    J = TCSteps.apply(x, S, S.zeros(3), 1, 1)
    assert J.grad_fn.overlap
    del J, x
    S.close()
    torch.cuda.empty_cache()
