"""Steps from face traces on meshes with curved elements against the chain of
dg_rk_stage, which evaluates both sides of a face from the states: the same
bits.  The curved set leaves its traces to the straight elements beside it; the
straight tiles leave out its outputs and traces.  Every order and form, the set
spread over tiles and workgroups, a moving wall, and every launch shape."""
import numpy as np
import pytest

import meshgen as mg
from tests.test_gpu_traces import _chain, _state, _torch

pytestmark = pytest.mark.gpu


def _curved_solver(nt, nr, growth, p, precision, theta):
    from paper_2508_17917_amd import Solver
    w = mg.physics_params(Re=100.0, M=0.2)
    return Solver(p, mg.ogrid(nt, nr, 0.5, 5.0, growth), precision=precision, penalty_mode=0, C_pen=1.0, theta=theta,
                  curved=mg.curve_wall, **w)


@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("p", range(1, 7))
def test_curved_steps_equal_the_stage_chain(p, precision):
    torch = _torch()
    from paper_2508_17917_amd import _lib as L
    s = _curved_solver(11, 5, 1.3, p, precision, 1.0 if p % 2 else 0.0)
    print("[gpu-case] curved traces p=%d precision=%d K=%d set=%d" % (
        p, precision, s.K, int((s.table("curved_slot") >= 0).sum())), flush=True)
    U = _state(torch, s, p)
    vw, nsteps, dt = (0.01, -0.03), 3, 1e-6
    want, K1w, Fw = _chain(torch, s, U, nsteps, dt, vw)
    assert bool(torch.isfinite(want).all()) and not torch.equal(want, U)
    for waves, grid in [(0, 0)] + [(w, g) for w in (2, 4) for g in range(4)]:
        s.set_tuning(waves, grid)
        got, K1 = U.clone(), torch.full_like(U, 7.0)
        F = torch.full((nsteps, 3), -1.0, dtype=torch.float64, device="cuda")
        s.rk_steps(got, K1, nsteps, dt, v_w=vw, force=F)
        assert torch.equal(got, want) and torch.equal(K1, K1w), (waves, grid, float((got - want).abs().max()))
        assert np.array_equal(F.cpu().numpy(), Fw), (waves, grid)
    got, K1 = U.clone(), torch.zeros_like(U)
    L.dg_rk_steps_noalloc(s.h, got, K1, nsteps, dt, vw)
    assert torch.equal(got, want) and torch.equal(K1, K1w)
    s.close()


@pytest.mark.parametrize("p,precision", [(2, 0), (4, 2), (6, 0)])
def test_curved_single_and_many_steps(p, precision):
    """More tiles than one round of the chip holds; one step (from traces from
    16,384 elements on) and several."""
    torch = _torch()
    s = _curved_solver(97, 89, 1.02, p, precision, 1.0)
    print("[gpu-case] curved traces p=%d precision=%d K=%d" % (p, precision, s.K), flush=True)
    U = _state(torch, s, p)
    for nsteps in (1, 4):
        want, K1w, _ = _chain(torch, s, U, nsteps, 1e-9, (0.0, 0.02))
        got, K1 = U.clone(), torch.full_like(U, 7.0)
        s.rk_steps(got, K1, nsteps, 1e-9, v_w=(0.0, 0.02))
        assert bool(torch.isfinite(want).all()) and not torch.equal(want, U)
        assert torch.equal(got, want) and torch.equal(K1, K1w), nsteps
    s.close()
