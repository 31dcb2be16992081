"""The set-up's backward-error check runs on the solves that the context's steps
use: with the line kernels it is theirs, at rounding like that of the factors
themselves but not the same number."""
import pytest

pytestmark = pytest.mark.gpu


def test_check_covers_the_line_solves(monkeypatch):
    from paper_1311_2481_amd import Solver
    errs = []
    # 2 to 32 lanes, full lines and lines with empty rows
    for n_r, m_theta, m_z in ((9, 8, 16), (16, 130, 128), (31, 8, 16), (40, 12, 20), (64, 64, 128), (101, 12, 20),
                              (200, 8, 16), (256, 8, 16)):
        for line in ("1", "0"):
            monkeypatch.setenv("TC_PC_LINE", line)
            S = Solver(n_r, m_theta, m_z, 0.6, 300.0, -50.0, 1e-5, alpha=0.5)
            errs.append(S.factor_backward_error())
            S.close()
        print(f"{n_r} x {m_theta} x {m_z}: line solves {errs[-2]:.2e}, the factors {errs[-1]:.2e}")
    assert all(0.0 < e < 1e-14 for e in errs)
    assert any(a != b for a, b in zip(errs[::2], errs[1::2]))
