"""The line kernels with 7 and 8 rows on a lane, which grids of many modes
keep, and with twice the lanes at the largest grids that take them: one step,
the solves and the adjoint step against the four-sweep kernels on the same
inputs.  Either form is held to ten times the one-ulp floor elsewhere, so they
may differ by twice that; the floor is that of the same nodes with few modes,
which are the worse conditioned."""
import numpy as np
import pytest

import tc_inputs
from oracle import adjoint as adj
from oracle import scheme
from gpu_common import floor_tol, make_pair, rel_l2, to_dev, to_host, twin_floor

pytestmark = pytest.mark.gpu

# lanes x rows: 2 x 7, 2 x 8, 4 x 7, 4 x 8, 8 x 7, 8 x 8; at the line, 4 x 5 and 16 x 5
GRIDS = [(14, 66, 250), (16, 66, 250), (27, 66, 126), (32, 66, 126), (55, 40, 104), (64, 40, 104),
         (13, 64, 256), (64, 32, 128)]


@pytest.mark.parametrize("n_r,m_theta,m_z", GRIDS)
def test_line_on_many_modes_matches_four_sweeps(n_r, m_theta, m_z, monkeypatch):
    def inputs(r, cfg):
        shape = (3, n_r, cfg.m_z, cfg.m_theta)
        u0 = tc_inputs.initial_state(r, cfg)
        up = u0 + 1e-3 * tc_inputs.random_state(shape, 61)
        up[:, 0], up[:, -1] = u0[:, 0], u0[:, -1]
        return [u0, up, u0 * 0.1] + [tc_inputs.random_state(shape, 62 + k, hermitian=False) for k in range(3)]

    def pair(m_t, m_zz):
        return make_pair("medium", n_r=n_r, m_theta=m_t, m_z=m_zz, dt=1e-6)

    S, P, cfg = pair(5, 14)
    S.close()
    u0, up, Np, a, b, c = inputs(P.r, cfg)
    what = {"u": lambda Q: scheme.step(Q, u0, up, Np)[0], "p": lambda Q: scheme.step(Q, u0, up, Np)[1],
            "adjoint": lambda Q: np.concatenate(adj.step_adjoint(Q, u0, a, b, c))}
    for kind in ("P", "Uz"):
        for trans in (0, 1):
            what[f"{kind} {trans}"] = lambda Q, kind=kind, trans=trans: Q.solve(kind, a[0], trans=trans)
    tol = {k: 2 * floor_tol(twin_floor(P, f, f(P))) for k, f in what.items()}

    got = []
    for line in (True, False):
        if not line:
            monkeypatch.setenv("TC_PC_LINE", "0")
        S, P, cfg = pair(m_theta, m_z)
        u0, up, Np, a, b, c = inputs(P.r, cfg)
        S.set_state(to_dev(u0), to_dev(up), to_dev(Np))
        S.step(1)
        u1, p1 = (to_host(x) for x in S.get_state())
        out = {"u": u1, "p": p1}
        out["adjoint"] = to_host(S.step_adjoint(to_dev(np.concatenate([u0, up])), to_dev(np.concatenate([a, b, c]))))
        for kind in ("P", "Uz"):
            for trans in (0, 1):
                out[f"{kind} {trans}"] = to_host(S.solve(kind, to_dev(a[0]), transposed=bool(trans)))
        got.append((out, S.memory_bytes()))
        S.close()
    assert got[0][1] > got[1][1]  # the line context holds its copy of the factors
    for k, t in tol.items():
        err = rel_l2(got[0][0][k], got[1][0][k])
        print(f"{n_r} x {m_theta} x {m_z} {k}: rel_l2 {err:.2e} (tolerance {t:.2e})")
        assert err <= t, k
