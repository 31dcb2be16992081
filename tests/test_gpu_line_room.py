"""Contexts short of memory for the line kernels' copy of the factors (TC_NO_ROOM
makes the named allocation count as failed): left out at tc_init; given up by
the first adjoint call; kept where giving it up does not help, and where a
captured graph may read it.  The line kernels and the four sweeps differ in
rounding, so equality bit for bit tells which of them ran."""
import numpy as np
import pytest

import tc_inputs
from gpu_common import to_dev, to_host

pytestmark = pytest.mark.gpu

N_R, M_THETA, M_Z = 40, 12, 20


def solver(monkeypatch, line=True, stream=None):
    from paper_1311_2481_amd import Solver
    cfg = tc_inputs.CONFIGS["medium"]
    with monkeypatch.context() as m:
        if not line:
            m.setenv("TC_PC_LINE", "0")
        return Solver(N_R, M_THETA, M_Z, cfg.eta, cfg.Re_i, cfg.Re_o, 1e-6, stream=stream)


def fields(S):
    cfg = tc_inputs.Config(tc_inputs.CONFIGS["medium"])
    cfg.update(n_r=N_R, m_theta=M_THETA, m_z=M_Z)
    u = to_dev(tc_inputs.initial_state(S.radial_nodes(), cfg))
    adj = to_dev(tc_inputs.random_state((9, N_R, M_Z, M_THETA), 81, hermitian=False))
    return u, adj


def stepped(S, u, n=2):
    S.set_state(u)
    S.step(n)
    return to_host(S.get_state(with_pressure=False))


def adjoint(S, u, adj):
    import torch
    return to_host(S.step_adjoint(torch.cat([u, u]), adj))


@pytest.fixture
def reference(monkeypatch):
    """(step, adjoint, bytes before the adjoint) of either kind of context."""
    out = []
    for line in (True, False):
        S = solver(monkeypatch, line)
        u, adj = fields(S)
        b = S.memory_bytes()
        out.append((stepped(S, u), adjoint(S, u, adj), b))
        S.close()
    (us, gs, bs), (uf, gf, bf) = out
    assert bs > bf and not np.array_equal(us, uf) and not np.array_equal(gs, gf)
    return out


def test_left_out_at_init(reference, monkeypatch):
    monkeypatch.setenv("TC_NO_ROOM", "lines")
    S = solver(monkeypatch)
    u, adj = fields(S)
    assert S.memory_bytes() == reference[1][2]
    assert np.array_equal(stepped(S, u), reference[1][0])
    assert np.array_equal(adjoint(S, u, adj), reference[1][1])
    S.close()


def test_given_up_by_the_first_adjoint_call(reference, monkeypatch):
    S = solver(monkeypatch)
    u, adj = fields(S)
    assert np.array_equal(stepped(S, u), reference[0][0])
    monkeypatch.setenv("TC_NO_ROOM", "adjoint")
    before = S.memory_bytes()
    g = adjoint(S, u, adj)
    monkeypatch.delenv("TC_NO_ROOM")
    assert np.array_equal(g, reference[1][1])
    full = solver(monkeypatch, line=False)
    adjoint(full, u, adj)
    assert before == reference[0][2] and S.memory_bytes() == full.memory_bytes()
    full.close()
    assert np.array_equal(stepped(S, u), reference[1][0])
    assert np.array_equal(adjoint(S, u, adj), reference[1][1])
    S.close()


def test_kept_where_giving_it_up_makes_no_room(reference, monkeypatch):
    from paper_1311_2481_amd import TcError
    S = solver(monkeypatch)
    u, adj = fields(S)
    S.set_state(u)
    S.step(1)
    monkeypatch.setenv("TC_NO_ROOM", "adjoint twice")
    with pytest.raises(TcError, match="ENOMEM"):
        adjoint(S, u, adj)
    monkeypatch.delenv("TC_NO_ROOM")
    assert S.memory_bytes() == reference[0][2]
    S.step(1)
    assert np.array_equal(to_host(S.get_state(with_pressure=False)), reference[0][0])
    assert np.array_equal(adjoint(S, u, adj), reference[0][1])
    S.close()


def test_kept_where_a_graph_reads_it(reference, monkeypatch):
    import torch
    from paper_1311_2481_amd import TcError
    s = torch.cuda.Stream()
    S = solver(monkeypatch, stream=s)
    with torch.cuda.stream(s):
        u, adj = fields(S)
        fwd = torch.cat([u, u])
        S.set_state(u)
        S.step(2)
        S.set_state(u)
    s.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        S.step(2)
    monkeypatch.setenv("TC_NO_ROOM", "adjoint")
    with pytest.raises(TcError, match="ENOMEM"):
        S.step_adjoint(fwd, adj)
    monkeypatch.delenv("TC_NO_ROOM")
    assert S.memory_bytes() == reference[0][2]
    for _ in range(3):
        with torch.cuda.stream(s):
            S.set_state(u)
            graph.replay()
            got = S.get_state(with_pressure=False)
        s.synchronize()
        assert np.array_equal(to_host(got), reference[0][0])
    with torch.cuda.stream(s):
        got = S.step_adjoint(fwd, adj)
    s.synchronize()
    assert np.array_equal(to_host(got), reference[0][1])
    S.close()
