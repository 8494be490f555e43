"""Periodic seams whose vertices are translates only to rounding, or only to the
matching tolerance (1e-8 of the mesh's extent): every element keeps the normals
of its own edges, on which its constant states' fluxes balance, and the steps
equal the chain of single stages although the two sides' normals do not negate
each other.  The geometry on the CPU, the steps on an MI355X.
"""
import os

import numpy as np
import pytest

import meshgen as mg

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2508_17917_amd", "libdgmi.so")


def _wavy(offset, n=(6, 5)):
    """A periodic square with bent seams, its right side off by up to `offset`."""
    mesh = mg.periodic_square(n[0], n[1], 2.0, 1.5)
    VX, VY = np.array(mesh["VX"]), np.array(mesh["VY"])
    right = VX > 2.0 - 1e-9
    VX, VY = VX + 0.1 * np.sin(2.0 * np.pi * VY / 1.5), VY + 0.05 * np.sin(np.pi * VX)
    VY[right] += offset * np.cos(40.0 * VX[right])
    return dict(mesh, VX=VX, VY=VY)


@pytest.mark.skipif(not os.path.exists(LIB), reason="libdgmi.so not built")
@pytest.mark.parametrize("offset", [0.0, 5e-9])
def test_elements_keep_their_own_normals(offset):
    from paper_2508_17917_amd import Solver
    mesh = _wavy(offset)
    s = Solver(2, mesh, device=False)
    geo = s.table("geo").reshape(-1, 16)
    x, y = mesh["VX"][mesh["EToV"]], mesh["VY"][mesh["EToV"]]
    nbr, nf = s.table("nbr").astype(int).reshape(-1, 3), s.table("nbr_face").astype(int).reshape(-1, 3)
    mismatch = 0.0
    for f in range(3):
        dx, dy = x[:, (f + 1) % 3] - x[:, f], y[:, (f + 1) % 3] - y[:, f]
        L = np.sqrt(dx * dx + dy * dy)
        assert np.abs(geo[:, 4 + 4 * f] - dy / L).max() <= 4e-16
        assert np.abs(geo[:, 5 + 4 * f] + dx / L).max() <= 4e-16
        for c in (4, 5):
            mismatch = max(mismatch, np.abs(geo[:, c + 4 * f] + geo[nbr[:, f], c + 4 * nf[:, f]]).max())
    # (the seam does what the case is for)
    assert mismatch > (1e-9 if offset else 0.0)
    s.close()


@pytest.mark.gpu
@pytest.mark.parametrize("offset", [0.0, 5e-9])
@pytest.mark.parametrize("precision", [0, 2, "overint"])
def test_steps_equal_the_stage_chain(precision, offset):
    from tests.test_gpu_traces import _chain, _solver, _state, _torch
    torch = _torch()
    print("[gpu-case] seam precision=%s offset=%g" % (precision, offset), flush=True)
    s = _solver(_wavy(offset), 3, precision, 1.0)
    U = _state(torch, s, 3)
    want, K1w, _ = _chain(torch, s, U, 3, 1e-5, (0.02, 0.01))
    got, K1 = U.clone(), torch.zeros_like(U)
    s.rk_steps(got, K1, 3, 1e-5, v_w=(0.02, 0.01))
    assert bool(torch.isfinite(want).all()) and not torch.equal(want, U)
    assert torch.equal(got, want) and torch.equal(K1, K1w)
    s.close()


@pytest.mark.gpu
def test_batch_with_such_a_mesh():
    """Among instances that traces serve: the batch's steps equal the chains."""
    from tests.test_gpu_traces import _batch_case, _chain, _torch
    torch = _torch()
    meshes = [_wavy(5e-9, (90, 70)), mg.ogrid(71, 53, 0.5, 8.0, 1.02)]
    print("[gpu-case] seam batch", flush=True)
    b, solvers, states = _batch_case(torch, (3, 2), meshes, 2, 5)
    assert sum(s.K for s in solvers) >= 16384
    dt, vw = np.full(2, 1e-6), np.zeros((2, 2))
    for i in range(2):
        b.set_state(i, states[i])
    b.rk_step(dt, vw)
    for i, s in enumerate(solvers):
        assert torch.equal(b.get_state(i), _chain(torch, s, states[i], 1, 1e-6, (0.0, 0.0))[0]), i
    b.close()
