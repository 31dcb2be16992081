"""The line kernels over their range of radial node counts: lines of 2 to 32
lanes with 5 to 8 rows each, full and with a partly or wholly empty last
lane, wall stencils that begin in the lane before the last; one step from
distinct u^i, u^{i-1}, N^{i-1}, the solves either way, and the adjoint step,
against the oracle within the one-ulp floors."""
import numpy as np
import pytest

import oracle
import tc_inputs
from oracle import adjoint as adj
from oracle import scheme
from gpu_common import floor_tol, make_pair, rel_l2, to_dev, to_host, twin_floor

pytestmark = pytest.mark.gpu

# n_r: smallest; (2 lanes, 8 rows) full; (4, 5) with 3 rows left; (4, 8) less one;
# (8, 5) full; (8, 6) with a last lane of 1; (8, 8) less one; (16, 5) with empty
# lanes; (16, 7); (16, 8) less three; (32, 5) with empty lanes; (32, 8) full
NODES = [9, 16, 17, 31, 40, 43, 63, 65, 101, 125, 129, 256]


@pytest.mark.parametrize("n_r", NODES)
def test_line_shapes_match_oracle(n_r):
    m_theta, m_z = 5, 14
    S, P, cfg = make_pair("medium", n_r=n_r, m_theta=m_theta, m_z=m_z, dt=1e-6)
    shape = (3, n_r, m_z, m_theta)
    u0 = tc_inputs.initial_state(P.r, cfg)
    up = u0 + 1e-3 * tc_inputs.random_state(shape, 31)
    up[:, 0], up[:, -1] = u0[:, 0], u0[:, -1]
    Np = oracle.nonlinear_rot(P, u0) + 0.1 * tc_inputs.random_state(shape, 32)

    def check(what, got, f):
        ref = f(P)
        err, floor = rel_l2(got, ref), twin_floor(P, f, ref)
        print(f"n_r={n_r} {what}: rel_l2 {err:.2e} (floor {floor:.2e})")
        assert err <= floor_tol(floor)

    S.set_state(to_dev(u0), to_dev(up), to_dev(Np))
    S.step(1)
    u1, p1 = (to_host(x) for x in S.get_state())
    check("u", u1, lambda Q: scheme.step(Q, u0, up, Np)[0])
    check("p", p1, lambda Q: scheme.step(Q, u0, up, Np)[1])
    rhs = tc_inputs.random_state((n_r, m_z, m_theta), 33, hermitian=False)
    for kind in ("P", "Up", "Um", "Uz"):
        for trans in (0, 1):
            out = S.empty(1).fill_(complex(7.0, -3.0))
            x = to_host(S.solve(kind, to_dev(rhs), out=out, transposed=bool(trans)))
            assert np.all(x[:, m_z // 2] == 0)
            check(f"{kind} trans={trans}", x, lambda Q: Q.solve(kind, rhs, trans=trans))
    a, b, c = (tc_inputs.random_state(shape, 34 + k, hermitian=False) for k in range(3))
    g = to_host(S.step_adjoint(to_dev(np.concatenate([u0, up])), to_dev(np.concatenate([a, b, c]))))
    for k in range(3):
        check(f"adjoint {k}", g[3 * k:3 * k + 3], lambda Q: adj.step_adjoint(Q, u0, a, b, c)[k])
    S.close()
