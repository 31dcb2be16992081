"""Calls that a change of kernel or route had made slower, each against another
call of the same library that does comparable work on the same grid, in one
process.  The comments give the ratio that was measured when it was slow."""
import time

import pytest

pytestmark = pytest.mark.gpu


def timed(f, repeats=5):
    """Seconds of a call, the least of several runs of at least 5 ms."""
    import torch
    f()
    torch.cuda.synchronize()
    t = time.perf_counter()
    f()
    torch.cuda.synchronize()
    n = max(3, int(5e-3 / max(time.perf_counter() - t, 1e-6)))
    best = float("inf")
    for _ in range(repeats):
        t = time.perf_counter()
        for _ in range(n):
            f()
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t) / n)
    return best


def solver(n_r, m_theta, m_z):
    from paper_1311_2481_amd import Solver
    return Solver(n_r, m_theta, m_z, 0.5, 1000.0, 0.0, 1e-9)


@pytest.mark.parametrize("n_r,m_theta,m_z,transposed", [(129, 100, 320, True), (200, 100, 300, True),
                                                        (100, 128, 380, True), (66, 128, 380, False)])
def test_solves_against_the_sweeps(n_r, m_theta, m_z, transposed, monkeypatch):
    # against the kernels of a context without the line copy: 1.85, 1.42, 1.29 and 1.10 times
    import torch
    t = []
    for line in ("1", "0"):
        monkeypatch.setenv("TC_PC_LINE", line)
        S = solver(n_r, m_theta, m_z)
        f = S.empty(1).fill_(complex(1.0, 0.5))
        x = S.empty(1)
        t.append([timed(lambda: S.solve(k, f, out=x, transposed=transposed)) for k in ("P", "Uz")])
        S.close()
        torch.cuda.synchronize()
    for k, a, b in zip(("P", "Uz"), *t):
        print(f"{n_r} x {m_theta} x {m_z} {k} transposed={transposed}: {a * 1e6:.0f} us, sweeps {b * 1e6:.0f} us")
        assert a <= 1.06 * b


@pytest.mark.parametrize("n_r,m_theta,m_z", [(9, 512, 1024), (10, 600, 1200)])
def test_diagnostics_of_large_planes(n_r, m_theta, m_z):
    # against the finite check, which reads the same velocity: 12.2 and 10.5 times its time
    S = solver(n_r, m_theta, m_z)
    d, f = timed(S.diag), timed(S.check_finite)
    print(f"{n_r} x {m_theta} x {m_z}: diagnostics {d * 1e6:.0f} us, finite check {f * 1e6:.0f} us")
    S.close()
    assert d <= 8 * f


@pytest.mark.parametrize("n_r,m_theta,m_z", [(9, 512, 1024), (16, 512, 1024)])
def test_set_up_of_the_line_copy(n_r, m_theta, m_z, monkeypatch):
    # what the line kernels' copy of the factors adds to a context's set-up, as
    # the rate at which its bytes are read and written: 1.4 and 1.5 TB/s
    best, held = {}, {}
    for _ in range(8):
        for line in ("1", "0"):
            monkeypatch.setenv("TC_PC_LINE", line)
            t = time.perf_counter()
            S = solver(n_r, m_theta, m_z)
            t = time.perf_counter() - t
            held[line] = S.memory_bytes()
            S.close()
            best[line] = min(best.get(line, t), t)
    rate = 2 * (held["1"] - held["0"]) / (best["1"] - best["0"])
    print(f"{n_r} x {m_theta} x {m_z}: set-up {best['1'] * 1e6:.0f} us, without the copy {best['0'] * 1e6:.0f} us, "
          f"{rate / 1e12:.2f} TB/s")
    assert rate >= 1.8e12
