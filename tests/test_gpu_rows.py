"""The kernels whose threads take groups of radial nodes of a mode (curl,
radial derivatives, the curl's adjoint, diagnostics) where a group or a
workgroup is partly filled, against the oracle: curl-type terms within the
one-ulp floors, diagnostics within their sums' rounding."""
import numpy as np
import pytest

import oracle
import tc_inputs
from oracle import adjoint as adj
from oracle import diagnostics as dg
from oracle import scheme
from gpu_common import floor_tol, make_pair, rel_l2, to_dev, to_host, twin_floor

pytestmark = pytest.mark.gpu

# n_r past a multiple of 4 by 0 to 3 (of 8 by 0 to 4), on 286 slots: one full
# workgroup and 30 threads; and on 8320 slots, more than the diagnostics'
# workgroups take in one round
SIZES = [(9, 13, 22), (10, 13, 22), (11, 13, 22), (12, 13, 22), (16, 64, 130), (17, 64, 130)]


@pytest.mark.parametrize("n_r,m_theta,m_z", SIZES)
def test_curl_rows(n_r, m_theta, m_z):
    from paper_1311_2481_amd import Solver
    S, P, cfg = make_pair("medium", n_r=n_r, m_theta=m_theta, m_z=m_z, dt=1e-6)
    shape = (3, n_r, m_z, m_theta)
    u = tc_inputs.initial_state(P.r, cfg) + 1e-3 * tc_inputs.random_state(shape, 41)

    def check(what, got, f):
        ref = f(P)
        err, floor = rel_l2(got, ref), twin_floor(P, f, ref)
        print(f"{n_r} x {m_theta} x {m_z} {what}: rel_l2 {err:.2e} (floor {floor:.2e})")
        assert err <= floor_tol(floor)

    check("omega x u", to_host(S.nonlinear(to_dev(u))), lambda Q: oracle.nonlinear_rot(Q, u))
    if m_z < 100:
        a, b, c = (tc_inputs.random_state(shape, 42 + k, hermitian=False) for k in range(3))
        g = to_host(S.step_adjoint(to_dev(np.concatenate([u, u])), to_dev(np.concatenate([a, b, c]))))
        check("adjoint", g[:3], lambda Q: adj.step_adjoint(Q, u, a, b, c)[0])
    S.close()
    S = Solver(n_r, m_theta, m_z, cfg.eta, cfg.Re_i, cfg.Re_o, cfg.dt, k_theta=cfg.k_theta, k_z=cfg.k_z,
               alpha=cfg.alpha, form="conv")
    check("u . grad u", to_host(S.nonlinear(to_dev(u))), lambda Q: oracle.nonlinear_conv(Q, u))
    S.close()


@pytest.mark.parametrize("n_r,m_theta,m_z", SIZES)
def test_diagnostics_rows(n_r, m_theta, m_z):
    S, P, cfg = make_pair("medium", n_r=n_r, m_theta=m_theta, m_z=m_z, dt=1e-6)
    u = tc_inputs.initial_state(P.r, cfg) + 1e-3 * tc_inputs.random_state((3, n_r, m_z, m_theta), 51)
    S.set_state(to_dev(u))
    d = S.diag()
    ref = dict(energy=dg.energy(P, u), perturbation_energy=dg.perturbation_energy(P, u),
               max_div=np.abs(scheme.div(P, u)[1:-1]).max(), slip=dg.wall_slip(P, u), cfl=dg.cfl_bound(P, u))
    # the divergence of this field is no cancellation, but its terms are
    # summed in another order
    a, b, r = P.bcast()
    ur = 0.5 * np.abs(u[0] + u[1])
    terms = (np.einsum("jk,ksn->jsn", np.abs(P.D1), ur) + ur / r + a * np.abs(u[0] - u[1]) / (2 * r)
             + np.abs(b * u[2]))
    tol = dict(max_div=1e-14 * terms[1:-1].max())
    for k, v in ref.items():
        print(f"{n_r} x {m_theta} x {m_z} {k}: gpu {d[k]:.15e} oracle {v:.15e}")
        assert abs(d[k] - v) <= tol.get(k, 1e-12 * abs(v)), k
    # a value that is not a number: the energies show it, the CFL bound is that
    # of the nodes behind it, the divergence that of the points without it
    j = n_r // 2
    w = u.copy()
    w[2, j, 1, 1] = complex(np.nan, 0.0)
    S.set_state(to_dev(w))
    d = S.diag()
    assert np.isnan(d["energy"]) and np.isnan(d["perturbation_energy"])
    tail = u.copy()
    tail[:, :j + 1] = 0
    assert abs(d["cfl"] - dg.cfl_bound(P, tail)) <= 1e-12 * d["cfl"]
    dv = np.abs(scheme.div(P, w)[1:-1])
    assert abs(d["max_div"] - np.nanmax(dv)) <= tol["max_div"]
    w[2, j, 1, 1] = complex(np.inf, 0.0)
    S.set_state(to_dev(w))
    d = S.diag()
    assert np.isinf(d["energy"]) and np.isinf(d["cfl"])
    S.close()
