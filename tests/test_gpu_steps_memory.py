"""Steps on contexts before and after they hold face traces and a second scratch
state (needs an MI355X): a first call recorded into a graph, which can allocate
neither, and over-integration switched on after nodal steps."""
import pytest

import meshgen as mg
from tests.test_gpu_traces import _chain, _solver, _state, _torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 2, "overint"])
@pytest.mark.parametrize("nsteps", [1, 2])
def test_first_call_captured(nsteps, precision):
    """The graph of a context's first steps, replayed on several states with
    eager steps of the same context in between, against the stage chain."""
    torch = _torch()
    print("[gpu-case] first call captured precision=%s nsteps=%d" % (precision, nsteps), flush=True)
    s = _solver(mg.ogrid(67, 64, 0.5, 8.0, 1.02), 3, precision, 1.0)
    vw, dt = (0.01, -0.03), 1e-6
    states = [_state(torch, s, k) for k in range(3)]
    want = [_chain(torch, s, u, nsteps, dt, vw)[0] for u in states]
    U, K1 = states[0].clone(), torch.zeros_like(states[0])
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        s.rk_steps(U, K1, nsteps, dt, v_w=vw, stream=torch.cuda.current_stream())
    for u, w in list(zip(states, want)) * 2:
        U.copy_(u)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(U, w)
        V = u.clone()
        s.rk_steps(V, torch.zeros_like(u), nsteps, dt, v_w=vw)
        torch.cuda.synchronize()
        assert torch.equal(V, w)
    s.close()


def test_overintegration_after_nodal_steps():
    torch = _torch()
    from paper_2508_17917_amd import _lib as L
    print("[gpu-case] over-integration switched on and off", flush=True)
    s = _solver(mg.ogrid(67, 64, 0.5, 8.0, 1.02), 3, 0, 1.0)
    u = _state(torch, s, 5)
    for on in (0, 1, 0, 1):
        L.dg_set_overintegration(s.h, on)
        want = _chain(torch, s, u, 2, 1e-6, (0.0, 0.02))[0]
        got = u.clone()
        s.rk_steps(got, torch.zeros_like(u), 2, 1e-6, v_w=(0.0, 0.02))
        assert torch.equal(got, want), on
    s.close()
