"""Both diagnostics entry points against the oracle: the eight values, over
grids whose slots take several rounds of the reducing workgroups, with partly
filled groups of radial nodes, and after a call on another grid has left its
partial sums in the same places."""
import ctypes

import numpy as np
import pytest

import tc_inputs
from oracle import diagnostics as dg
from oracle import scheme
from gpu_common import make_pair, node_jitter_twin, to_dev

pytestmark = pytest.mark.gpu

NAMES = ["energy", "perturbation_energy", "max_div", "slip", "cfl", "steps", "nu_inner", "nu_outer"]


def _call(S, fn):
    out = np.full(8, -1.0)
    assert fn(S.ctx, out.ctypes.data_as(ctypes.POINTER(ctypes.c_double))) == 0
    return dict(zip(NAMES, out))


def expected(P, u):
    """{name: (value, tolerance)}: sums to 1e-12 of themselves; the divergence and
    the wall torques, which cancel and whose D1 weights carry the rounding of the
    nodes, to ten times what moving the nodes by an ulp changes, and no less than
    1e-14 of the sum of their terms."""
    ref = dict(energy=dg.energy(P, u), perturbation_energy=dg.perturbation_energy(P, u), slip=dg.wall_slip(P, u),
               cfl=dg.cfl_bound(P, u))
    ref = {k: (v, 1e-12 * abs(v)) for k, v in ref.items()}
    a, b, r = P.bcast()
    terms = (np.einsum("jk,ksn->jsn", np.abs(P.D1), 0.5 * np.abs(u[0] + u[1])) + 0.5 * np.abs(u[0] + u[1]) / r
             + a * np.abs(u[0] - u[1]) / (2 * r) + np.abs(b * u[2]))
    mean = np.abs(0.5 * (u[0, :, 0, 0].imag - u[1, :, 0, 0].imag)) / P.r
    torque = abs(2 * P.eta * (P.Re_i - P.eta * P.Re_o) / ((1 - P.eta) * (1 - P.eta ** 2)))
    f = {"max_div": (lambda Q: np.abs(scheme.div(Q, u)[1:-1]).max(), terms[1:-1].max()),
         "nu_inner": (lambda Q: dg.quasi_nusselt(Q, u)[0], P.r[0] ** 3 * (np.abs(P.D1[0]) @ mean) / torque),
         "nu_outer": (lambda Q: dg.quasi_nusselt(Q, u)[1], P.r[-1] ** 3 * (np.abs(P.D1[-1]) @ mean) / torque)}
    twins = [node_jitter_twin(P, s) for s in (1, 2, 3)]
    for k, (fn, size) in f.items():
        ref[k] = (fn(P), max(10 * max(abs(fn(Q) - fn(P)) for Q in twins), 1e-14 * size))
    return ref


@pytest.mark.parametrize("n_r,m_theta,m_z", [(9, 96, 256), (20, 64, 160), (75, 16, 40), (9, 2, 4)])
def test_diagnostics_match_oracle(n_r, m_theta, m_z):
    S, P, cfg = make_pair("medium", n_r=n_r, m_theta=m_theta, m_z=m_z, dt=1e-6)
    T, Q, other = make_pair("small")
    u = tc_inputs.initial_state(P.r, cfg) + 1e-3 * tc_inputs.random_state((3, n_r, m_z, m_theta), 91)
    T.set_state(to_dev(tc_inputs.initial_state(Q.r, other)))
    S.set_state(to_dev(u))
    ref = expected(P, u)
    for fn in (S.lib.tc_get_diag, S.lib.tc_get_diag_noalloc):
        _call(T, fn)
        d = _call(S, fn)
        assert d["steps"] == 0
        for k, (v, tol) in ref.items():
            print(f"{n_r} x {m_theta} x {m_z} {k}: gpu {d[k]:.15e} oracle {v:.15e} (tolerance {tol:.1e})")
            assert abs(d[k] - v) <= tol, k
    S.close()
    T.close()
