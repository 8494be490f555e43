"""A non-finite value stays where the method carries it (needs an MI355X).

One stage spreads a NaN or an infinity to the element's face neighbours and no
further.  The steps from face traces work tile after tile in the same LDS, and
a batch instance after instance, so a value that one tile leaves behind must
not reach the next one's products: a mesh with one bad element ends with the
finite values, and the finite places, of the chain of dg_rk_stage, and the
other instances of a batch with one that diverged keep the bits of their own
chains.  Every order and every form with traces, several tiles per wave.
"""
import numpy as np
import pytest

import meshgen as mg
from tests.test_gpu_curved_traces import _curved_solver
from tests.test_gpu_traces import _batch_case, _chain, _solver, _state, _torch

pytestmark = pytest.mark.gpu

# what becomes of node 0 of the element
BAD = {
    "nan": lambda u: u.__setitem__((0, 0), float("nan")),
    "inf": lambda u: u.__setitem__((3, 0), float("inf")),
    # the density so small that mu / rho, and with it the norm, overflows
    "tiny": lambda u: u.__setitem__((slice(None), 0), u.new_tensor([1e-313, 0.0, 0.0, 2.5e-313])),
}


def _same(torch, a, b):
    fa, fb = torch.isfinite(a), torch.isfinite(b)
    return torch.equal(fa, fb) and torch.equal(torch.where(fa, a, 0.0), torch.where(fb, b, 0.0))


def _steps_against_chain(torch, s, U, bad, shapes, spreads=True):
    vw, nsteps, dt = (0.01, -0.03), 2, 1e-7
    V = U.clone()
    for k, kind in bad:
        BAD[kind](V[k])
    want, K1w, _ = _chain(torch, s, V, nsteps, dt, vw)
    ok = torch.isfinite(want).all(dim=2).all(dim=1)
    assert int(ok.sum()) > s.K // 2 and (spreads is False or not bool(ok.all()))
    for waves, grid in shapes:
        s.set_tuning(waves, grid)
        got, K1 = V.clone(), torch.full_like(V, 7.0)
        s.rk_steps(got, K1, nsteps, dt, v_w=vw)
        assert _same(torch, got, want) and _same(torch, K1, K1w), (
            waves, grid, int((~torch.isfinite(got)).sum()), int((~torch.isfinite(want)).sum()))


@pytest.mark.parametrize("kind", sorted(BAD))
@pytest.mark.parametrize("precision", [0, 1, 2, "overint"])
@pytest.mark.parametrize("p", range(1, 7))
def test_a_bad_element_stays_within_the_stencil(p, precision, kind):
    """8,576 elements, three tiles a wave or as many as a persistent grid has."""
    torch = _torch()
    print("[gpu-case] non-finite %s p=%d precision=%s" % (kind, p, precision), flush=True)
    s = _solver(mg.ogrid(67, 64, 0.5, 8.0, 1.02), p, precision, 1.0)
    # (the over-integrated points are not the nodes: there the tiny density is none)
    _steps_against_chain(torch, s, _state(torch, s, p), [(s.K // 2 + 1, kind)], [(4, 3), (2, 3), (4, 0)],
                         spreads=not (precision == "overint" and kind == "tiny"))
    s.close()


@pytest.mark.parametrize("kind", ["nan", "inf"])
@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("p", range(1, 7))
def test_a_bad_element_of_the_curved_set(p, precision, kind):
    """The bad element in the set that other waves advance (the first wall
    element, and a face neighbour of another): the straight tiles leave its
    outputs and traces out, and nothing of it reaches the elements after it.
    The chain is compared on the elements that stay finite as well as by where
    they do."""
    torch = _torch()
    print("[gpu-case] non-finite curved %s p=%d precision=%d" % (kind, p, precision), flush=True)
    s = _curved_solver(67, 64, 1.02, p, precision, 1.0)
    curved = np.flatnonzero(s.table("curved_slot") >= 0)
    bad = [(int(curved[0]), kind), (int(curved[-1]), kind)]
    _steps_against_chain(torch, s, _state(torch, s, p), bad, [(4, 3), (2, 3), (4, 0)])
    s.close()


@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("p", range(1, 7))
def test_a_diverged_instance_leaves_the_others_alone(p, precision):
    """Four instances of one order, the first with a NaN element every 16, the
    third with an infinite one, laid out so that a wave's tiles run from a bad
    instance into a good one."""
    torch = _torch()
    print("[gpu-case] non-finite batch p=%d precision=%d" % (p, precision), flush=True)
    meshes = [mg.ogrid(a, b, 0.5, 8.0, 1.02) for a, b in ((67, 31), (127, 111), (61, 33), (113, 121))]
    b, solvers, states = _batch_case(torch, (p,) * 4, meshes, precision, 31)
    for k in range(0, solvers[0].K, 16):
        BAD["nan"](states[0][k])
    for k in range(0, solvers[2].K, 16):
        BAD["inf"](states[2][k])
    dt, vw = np.full(4, 1e-7), np.array([[0.0, 0.01 * i] for i in range(4)])
    want = [_chain(torch, s, u, 1, 1e-7, tuple(v))[0] for s, u, v in zip(solvers, states, vw)]
    for mode, waves, grid in [(0, 4, 0), (1, 4, 0), (1, 2, 0)]:
        b.configure(mode, waves, grid, True)
        for i in range(4):
            b.set_state(i, states[i])
        b.rk_step(dt, vw)
        for i in (1, 3):
            assert bool(torch.isfinite(want[i]).all())
            assert torch.equal(b.get_state(i), want[i]), (mode, waves, i, int((~torch.isfinite(b.get_state(i))).sum()))
        for i in (0, 2):
            assert _same(torch, b.get_state(i), want[i]), (mode, waves, i)
    b.close()
