"""The stage from face traces against the stage from the neighbours' states
(needs an MI355X).

dg_rk_step and dg_rk_steps leave each stage's face traces to the next one;
dg_rk_stage rebuilds the neighbours' gradients from their states.  The two
give the same bits: the same operations in the same order, the neighbour's
normal the own one negated, and matrix-core products that equal chains of
fused multiply-adds.  Cases: every order and form, a ragged O-grid with wall
(at rest and moving), far field and NIPG/IIPG/SIPG, a periodic square whose
seam vertices are not representable, two elements that are each other's only
neighbours, an element count below one tile, and every launch shape.
"""
import numpy as np
import pytest

import meshgen as mg

pytestmark = pytest.mark.gpu

A = (0.0, -567301805773.0 / 1357537059087.0, -2404267990393.0 / 2016746695238.0,
     -3550918686646.0 / 2091501179385.0, -1275806237668.0 / 842570457699.0)
B = (1432997174477.0 / 9575080441755.0, 5161836677717.0 / 13612068292357.0,
     1720146321549.0 / 2090206949498.0, 3134564353537.0 / 4481467310338.0,
     2277821191437.0 / 14882151754819.0)

MESHES = {
    "ogrid": lambda: mg.ogrid(7, 5, 0.5, 5.0, 1.3),            # 70 elements
    "periodic": lambda: mg.periodic_square(7, 3, 1.0 / 3.0, 0.7, 0.1, 0.2),
    "two": lambda: mg.periodic_square(1, 1, 10.0, 10.0),
}


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _solver(mesh, p, precision, theta):
    from paper_2508_17917_amd import Solver
    w = mg.physics_params(Re=100.0, M=0.2)
    return Solver(p, mesh, precision=precision, penalty_mode=0, C_pen=1.0, theta=theta, **w)


def _state(torch, s, seed):
    U = mg.noisy_free_stream((4, s.Np, s.K), mg.free_stream(0.2), mg.rng_for(1, salt=seed), amp=1e-2)
    return torch.from_numpy(np.ascontiguousarray(np.transpose(U, (2, 0, 1)))).cuda()


def _chain(torch, s, U, nsteps, dt, vw):
    """nsteps steps of dg_rk_stage, the force after each."""
    Ua, Ub, K1, F = U.clone(), torch.empty_like(U), torch.zeros_like(U), []
    for _ in range(nsteps):
        for a, b in zip(A, B):
            s.rk_stage(Ua, Ub, K1, a, b, dt, v_w=vw)
            Ua, Ub = Ub, Ua
        F.append(s.force(Ua, v_w=vw))
    return Ua, K1, np.array(F)


@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("p", range(1, 7))
@pytest.mark.parametrize("name", sorted(MESHES))
def test_steps_equal_the_stage_chain(name, p, precision):
    torch = _torch()
    theta, vw = {"ogrid": (1.0, (0.01, -0.03)), "periodic": (0.0, (0.02, 0.01)), "two": (-1.0, (0.0, 0.0))}[name]
    print("[gpu-case] traces %s p=%d precision=%d" % (name, p, precision), flush=True)
    s = _solver(MESHES[name](), p, precision, theta)
    U = _state(torch, s, p)
    nsteps, dt = 3, 1e-5
    want, K1w, Fw = _chain(torch, s, U, nsteps, dt, vw)
    assert bool(torch.isfinite(want).all()) and not torch.equal(want, U)
    shapes = [(0, 0)] + ([(w, g) for w in (2, 4) for g in range(4)] if name == "ogrid" else [])
    for waves, grid in shapes:
        s.set_tuning(waves, grid)
        got, K1 = U.clone(), torch.full_like(U, 7.0)
        F = torch.full((nsteps, 3), -1.0, dtype=torch.float64, device="cuda")
        s.rk_steps(got, K1, nsteps, dt, v_w=vw, force=F)
        assert torch.equal(got, want) and torch.equal(K1, K1w), (waves, grid, float((got - want).abs().max()))
        assert np.array_equal(F.cpu().numpy(), Fw), (waves, grid)
    one, K1 = U.clone(), torch.zeros_like(U)
    for _ in range(nsteps):
        s.rk_step(one, K1, dt, v_w=vw)
    assert torch.equal(one, want) and torch.equal(K1, K1w)
    s.close()


@pytest.mark.parametrize("p,precision,n", [(3, 2, 313), (4, 0, 271), (4, 2, 263), (5, 2, 235), (6, 0, 187)])
def test_streaming_steps_equal_the_stage_chain(p, precision, n):
    """Just beyond the last-level cache (the stage's arrays over 256 MB), where
    the launch stores whole lines past it; the element count is no multiple of
    the tile."""
    torch = _torch()
    mesh = mg.ogrid(n, n - 2, 0.5, 30.0, 1.01)
    K, size = 2 * n * (n - 2), 4 if precision == 2 else 8
    assert K % (3 if p >= 5 else 4) != 0 and K * (96 * ((p + 1) * (p + 2) // 2) + 24 * size * (p + 1) + 128) > 256 << 20
    print("[gpu-case] streaming traces p=%d precision=%d K=%d" % (p, precision, K), flush=True)
    s = _solver(mesh, p, precision, 1.0)
    U = _state(torch, s, p)
    want, K1w, Fw = _chain(torch, s, U, 2, 1e-8, (0.0, 0.02))
    got, K1 = U.clone(), torch.full_like(U, 7.0)
    F = torch.full((2, 3), -1.0, dtype=torch.float64, device="cuda")
    s.rk_steps(got, K1, 2, 1e-8, v_w=(0.0, 0.02), force=F)
    assert bool(torch.isfinite(want).all()) and not torch.equal(want, U)
    assert torch.equal(got, want) and torch.equal(K1, K1w)
    assert np.array_equal(F.cpu().numpy(), Fw)
    s.close()
