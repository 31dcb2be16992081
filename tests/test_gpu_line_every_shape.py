"""Every shape of the line kernels (2 to 32 lanes of 5 to 8 rows) against the
oracle: one step from distinct u^i, u^{i-1}, N^{i-1}, solves either way and the
adjoint step, within the one-ulp floors.  The shape that a grid gets is read off
the size of its copy of the factors, so a grid that a change of the rule moves
to another shape fails here; and the grids that the four sweeps keep, with the
kernels that only they use."""
import numpy as np
import pytest

import oracle
import tc_inputs
from oracle import adjoint as adj
from oracle import scheme
from gpu_common import floor_tol, make_pair, rel_l2, to_dev, to_host, twin_floor

pytestmark = pytest.mark.gpu

# lanes, rows, then the grid.  A grid of few modes takes twice the lanes where
# that saves two rows, so 7 and 8 rows on up to 8 lanes need many
SHAPES = [(2, 5, 10, 5, 14), (2, 6, 11, 5, 14), (2, 7, 14, 64, 258), (2, 8, 15, 64, 258),
          (4, 5, 18, 5, 14), (4, 6, 23, 5, 14), (4, 7, 27, 64, 130), (4, 8, 31, 64, 130),
          (8, 5, 33, 5, 14), (8, 6, 45, 5, 14), (8, 7, 53, 32, 130), (8, 8, 60, 32, 130),
          (16, 5, 72, 5, 14), (16, 6, 90, 5, 14), (16, 7, 105, 5, 14), (16, 8, 120, 5, 14),
          (32, 5, 140, 5, 14), (32, 6, 180, 5, 14), (32, 7, 210, 5, 14), (32, 8, 250, 5, 14)]


def places(S):
    """lanes x rows of a context's lines: the copy holds 36 doubles for each place
    and mode and 24 more for each place."""
    n, rest = divmod(S.line_copy_bytes(), 8 * (36 * S.m_theta * (S.m_z // 2) + 24))
    assert rest == 0
    return n


def inputs(r, cfg, n_r):
    shape = (3, n_r, cfg.m_z, cfg.m_theta)
    u0 = tc_inputs.initial_state(r, cfg)
    up = u0 + 1e-3 * tc_inputs.random_state(shape, 31)
    up[:, 0], up[:, -1] = u0[:, 0], u0[:, -1]
    return [u0, up, u0 * 0.1] + [tc_inputs.random_state(shape, 32 + k, hermitian=False) for k in range(3)]


def quantities(u0, up, Np, a, b, c):
    what = {"u": lambda Q: scheme.step(Q, u0, up, Np)[0], "p": lambda Q: scheme.step(Q, u0, up, Np)[1],
            "adjoint": lambda Q: np.concatenate(adj.step_adjoint(Q, u0, a, b, c))}
    for kind in ("P", "Um"):
        for trans in (0, 1):
            what[f"{kind} trans={trans}"] = lambda Q, kind=kind, trans=trans: Q.solve(kind, a[0], trans=trans)
    return what


def results(S, u0, up, Np, a, b, c):
    S.set_state(to_dev(u0), to_dev(up), to_dev(Np))
    S.step(1)
    u1, p1 = (to_host(x) for x in S.get_state())
    out = {"u": u1, "p": p1,
           "adjoint": to_host(S.step_adjoint(to_dev(np.concatenate([u0, up])), to_dev(np.concatenate([a, b, c]))))}
    for kind in ("P", "Um"):
        for trans in (0, 1):
            out[f"{kind} trans={trans}"] = to_host(S.solve(kind, to_dev(a[0]), transposed=bool(trans)))
    return out


def few_modes_floor(n_r):
    """The floors on the same nodes with few modes, which are the worse
    conditioned and which the oracle's twins can afford."""
    S, P, cfg = make_pair("medium", n_r=n_r, m_theta=5, m_z=14, dt=1e-6)
    S.close()
    return {k: floor_tol(twin_floor(P, f, f(P))) for k, f in quantities(*inputs(P.r, cfg, n_r)).items()}


def check(n_r, m_theta, m_z, expected):
    tol = few_modes_floor(n_r)
    S, P, cfg = make_pair("medium", n_r=n_r, m_theta=m_theta, m_z=m_z, dt=1e-6)
    assert places(S) == expected
    x = inputs(P.r, cfg, n_r)
    got = results(S, *x)
    S.close()
    for k, f in quantities(*x).items():
        err = rel_l2(got[k], f(P))
        print(f"{n_r} x {m_theta} x {m_z} {k}: rel_l2 {err:.2e} (tolerance {tol[k]:.2e})", flush=True)
        assert err <= tol[k], k


@pytest.mark.parametrize("lanes,rows,n_r,m_theta,m_z", SHAPES)
def test_every_line_shape_matches_oracle(lanes, rows, n_r, m_theta, m_z):
    check(n_r, m_theta, m_z, lanes * rows)


def test_four_sweeps_by_rule_match_oracle():
    # more nodes than 32 lanes of 8 rows
    check(260, 5, 14, 0)


def test_fused_curl_of_the_sweeps_matches_standalone(monkeypatch):
    # from 65536 distinct modes the last of the four sweeps also forms the curl of
    # the new velocity: two steps in one call against one step, a reload of the
    # state, which discards that curl, and another
    from paper_1311_2481_amd import Solver
    monkeypatch.setenv("TC_PC_LINE", "0")
    args = (16, 128, 1040, 0.6, 300.0, -50.0, 1e-4)
    cfg = tc_inputs.Config(n_r=16, m_theta=128, m_z=1040, eta=0.6, Re_i=300.0, Re_o=-50.0, dt=1e-4, amp=0.05,
                           envelope="k53", seed=9, k_theta=1.0, k_z=1.0, alpha=0.0)
    S = Solver(*args)
    assert places(S) == 0
    u0 = to_dev(tc_inputs.initial_state(S.radial_nodes(), cfg))
    S.set_state(u0)
    S.step(2)
    ua, pa = (to_host(x) for x in S.get_state())
    S.set_state(u0)
    S.step(1)
    u1 = S.get_state(with_pressure=False)
    S.set_state(u1, *S.get_history())
    S.step(1)
    ub, pb = (to_host(x) for x in S.get_state())
    S.close()
    eu, ep = rel_l2(ua, ub), rel_l2(pa, pb)
    print(f"fused vs standalone curl after two steps: u {eu:.2e}, p {ep:.2e}")
    assert eu < 1e-14 and ep < 1e-13
