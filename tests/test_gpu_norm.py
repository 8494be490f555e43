"""The largest singular value of the normal viscous matrix over states that take
each way through its iteration (four Newton steps, a fifth, the closed form):
the CFL bound, dominated by it at a large C_grad, against the oracle's dense
singular values at the bound of the CFL parity tests, 1e-12 relative."""
import numpy as np
import pytest

import meshgen as mg
from oracle.cfl import CFLOracle
from tests.oracle_helpers import build
from tests.test_gpu_parity import _say, _solver, _to_dev, _torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Pr", [0.72, 1.0, 3.0])
@pytest.mark.parametrize("e_lo,e_hi,speed", [(1.7, 1.9, 0.2), (0.9, 1.3, 0.4), (0.3, 0.9, 1.0), (0.05, 0.3, 0.1)])
def test_norm_over_the_iterations_ways(e_lo, e_hi, speed, Pr):
    """Total energies down to where the two largest eigenvalues meet; one
    element's worth of states at a time decides the bound, so each of several
    draws tests another few."""
    torch = _torch()
    mesh = mg.periodic_square(1, 1, 1.0, 1.0)
    dg = build(mesh, 3, Pr=Pr)
    c = CFLOracle(dg.mesh, dg.phys)
    s = _solver(mesh, 3, dg.phys)
    _say("norm e=%g..%g Pr=%g" % (e_lo, e_hi, Pr))
    rng = np.random.default_rng(5)
    for _ in range(20):
        shape = dg.mesh.x.shape
        v = rng.uniform(-speed, speed, (2,) + shape)
        rho = rng.uniform(0.5, 2.0, shape)
        E = rng.uniform(e_lo, e_hi, shape) + 0.5 * (v ** 2).sum(0)
        U = np.stack([rho, rho * v[0], rho * v[1], rho * E])
        want, _ = c.time_step(U, (0.0, 0.0), C_grad=100.0)
        lam, _ = s.cfl_time_step(_to_dev(torch, U), C_grad=100.0)
        assert abs(lam - want) <= 1e-12 * want, (lam, want)
    s.close()
