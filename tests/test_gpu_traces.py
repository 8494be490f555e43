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
    oi = precision == "overint"
    return Solver(p, mesh, precision=0 if oi else precision, overintegration=oi, penalty_mode=0, C_pen=1.0,
                  theta=theta, **w)


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


@pytest.mark.parametrize("precision", [0, 1, 2, "overint"])
@pytest.mark.parametrize("p", range(1, 7))
@pytest.mark.parametrize("name", sorted(MESHES))
def test_steps_equal_the_stage_chain(name, p, precision):
    torch = _torch()
    theta, vw = {"ogrid": (1.0, (0.01, -0.03)), "periodic": (0.0, (0.02, 0.01)), "two": (-1.0, (0.0, 0.0))}[name]
    print("[gpu-case] traces %s p=%d precision=%s" % (name, p, precision), flush=True)
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


def _batch_case(torch, orders, meshes, precision, seed):
    from paper_2508_17917_amd.solver import Batch
    solvers = [_solver(m, p, precision, 1.0) for p, m in zip(orders, meshes)]
    states = [_state(torch, s, seed + i) for i, s in enumerate(solvers)]
    return Batch(solvers), solvers, states


@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("orders,sizes", [
    ((4, 1, 6, 4), ((71, 53), (41, 60), (37, 61), (7, 5))),        # tiles of 4, 8 and 3, two instances of one order
    ((2, 3, 5), ((61, 61), (47, 51), (45, 53))),
])
def test_batch_equals_the_stage_chain(orders, sizes, precision):
    """A batch large enough for traces (16,384 elements or more), in every
    launch plan, on its own and on the caller's states, with the wall velocity
    and time step changing between steps, against dg_rk_stage chains."""
    torch = _torch()
    print("[gpu-case] batch traces orders=%s precision=%d" % (orders, precision), flush=True)
    meshes = [mg.ogrid(a, b, 0.5, 8.0, 1.02) for a, b in sizes]
    assert sum(2 * a * b for a, b in sizes) >= 16384
    b, solvers, states = _batch_case(torch, orders, meshes, precision, 3)
    n = len(solvers)
    dts = [np.array([1e-6 * (1 + i + k) for i in range(n)]) for k in range(2)]
    vws = [np.array([[0.01 * i, 0.02 * (k + 1)] for i in range(n)]) for k in range(2)]
    want = []
    for i, s in enumerate(solvers):
        U = states[i]
        for k in range(2):
            U, K1, _ = _chain(torch, s, U, 1, float(dts[k][i]), tuple(vws[k][i]))
        want.append((U, K1))
    for mode, waves, grid, graph in [(0, 4, 0, 1), (0, 2, 1, 0), (1, 4, 0, 1), (1, 2, 0, 1), (1, 4, 1, 0)]:
        b.configure(mode, waves, grid, bool(graph))
        for i in range(n):
            b.set_state(i, states[i])
        for k in range(2):
            b.rk_step(dts[k], vws[k])
        for i in range(n):
            assert torch.equal(b.get_state(i), want[i][0]), (mode, waves, grid, graph, i)
    Us = [u.clone() for u in states]
    K1s = [torch.full_like(u, 7.0) for u in states]
    for k in range(2):
        b.rk_step_states(Us, K1s, dts[k], vws[k])
    for i in range(n):
        assert torch.equal(Us[i], want[i][0]) and torch.equal(K1s[i], want[i][1]), i
    b.close()


def test_streaming_batch_equals_the_stage_chain():
    """Beyond the last-level cache: orders 2 (seven-element tiles) and 6."""
    torch = _torch()
    meshes = [mg.ogrid(331, 171, 0.5, 30.0, 1.01), mg.ogrid(131, 143, 0.5, 30.0, 1.01)]
    b, solvers, states = _batch_case(torch, (2, 6), meshes, 0, 11)
    K2, K6 = (s.K for s in solvers)
    assert K2 * 1280 + K6 * 4160 > 256 << 20 and K2 % 7 and K6 % 3
    print("[gpu-case] streaming batch traces K=%d, %d" % (K2, K6), flush=True)
    dt, vw = np.array([1e-7, 2e-7]), np.array([[0.0, 0.02], [0.01, 0.0]])
    for i in range(2):
        b.set_state(i, states[i])
    for mode in (0, 1):
        b.configure(mode, 4, 0, True)
        for i in range(2):
            b.set_state(i, states[i])
        b.rk_step(dt, vw)
        for i, s in enumerate(solvers):
            U, _, _ = _chain(torch, s, states[i], 1, float(dt[i]), tuple(vw[i]))
            assert torch.equal(b.get_state(i), U), (mode, i)
    b.close()


def test_batch_traces_follow_the_states():
    """The traces a step leaves serve the next one only while the states are
    those it left: one state replaced, steps on the caller's states and the
    autotuner in between, the wall velocity changing every step."""
    torch = _torch()
    sizes = ((71, 53), (41, 60), (37, 61), (7, 5))
    meshes = [mg.ogrid(a, c, 0.5, 8.0, 1.02) for a, c in sizes]
    b, solvers, states = _batch_case(torch, (4, 3, 6, 4), meshes, 2, 21)
    n = len(solvers)
    dt = np.full(n, 1e-6)
    vw = lambda k: np.array([[0.0, 0.01 * (k + i)] for i in range(n)])  # noqa: E731
    cur = [u.clone() for u in states]
    for i in range(n):
        b.set_state(i, cur[i])
    for k in range(5):
        if k == 2:
            cur[1] = states[1] * 1.001
            b.set_state(1, cur[1])
        if k == 3:
            b.autotune(reps=1)
        if k == 4:
            b.rk_step_states([u.clone() for u in states], [torch.zeros_like(u) for u in states], dt, vw(9))
            for i in range(n):
                b.set_state(i, cur[i])
        b.rk_step(dt, vw(k))
        for i, s in enumerate(solvers):
            cur[i] = _chain(torch, s, cur[i], 1, 1e-6, tuple(vw(k)[i]))[0]
            assert torch.equal(b.get_state(i), cur[i]), (k, i)
    b.close()
