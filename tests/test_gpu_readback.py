"""GPU tests of the results that kernels leave in pinned memory and of the
buffers an odd number of stages runs through: the CFL bound's maximum wherever
its element lies among the reducing workgroups, the host's sum of the force
partials, and odd steps on both sides of the size that gets a second scratch
state."""
import numpy as np
import pytest

import meshgen as mg
from tests.test_gpu_traces import _chain, _solver, _state, _torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nt,nr", [(1, 1), (16, 8), (43, 3), (33, 17)])
def test_cfl_maximum_in_every_workgroup(nt, nr):
    """256 elements per workgroup (2, 256, 258 and 1122 elements).  A faster,
    denser state in one element raises the bound of the whole mesh to that
    element's own, whichever workgroup has it: the same bits at every place of a
    uniform periodic mesh.  A NaN is refused from every place, and the bound of
    the state without it comes back afterwards."""
    torch = _torch()
    from paper_2508_17917_amd import _lib as L
    s = _solver(mg.periodic_square(nt, nr, float(nt), float(nr)), 2, 0, 1.0)
    print("[gpu-case] cfl workgroups K=%d" % s.K, flush=True)
    U = torch.from_numpy(np.array(mg.free_stream(0.2))).cuda()[None, :, None].expand(s.K, 4, s.Np).contiguous()
    base, _ = s.cfl_time_step(U)
    for k in sorted({0, s.K // 2, s.K - 2 - s.K % 2, s.K - 2}):
        V = U.clone()
        V[k, 3] *= 4.0
        lam, dt = s.cfl_time_step(V, C_cfl=0.5)
        assert lam > 1.5 * base and dt == 0.5 / lam
        # the same element type (its place within the square) everywhere: K - 2 and 0 are both even
        if k == 0:
            first = lam
        elif k % 2 == 0:
            assert abs(lam - first) <= 1e-12 * first, (k, lam, first)
        V[k, 0, 0] = float("nan")
        with pytest.raises(L.DGError):
            s.cfl_time_step(V)
        assert s.cfl_time_step(U)[0] == base
    s.close()


@pytest.mark.parametrize("nt,nr", [(1, 2), (16, 3), (43, 4)])
def test_force_of_every_partial_count(nt, nr):
    """One wall node block, an exact number of blocks and a ragged one: the
    host's sum equals the device's, bit for bit."""
    torch = _torch()
    s = _solver(mg.ogrid(max(nt, 3), nr, 0.5, 5.0, 1.3), 3, 0, 1.0)
    U = _state(torch, s, 3)
    dev = torch.zeros(3, dtype=torch.float64, device="cuda")
    from paper_2508_17917_amd import _lib as L
    L.dg_force_device(s.h, U, dev, (0.01, -0.02))
    for _ in range(2):
        assert np.array_equal(s.force(U, v_w=(0.01, -0.02)), dev.cpu().numpy())
    s.close()


@pytest.mark.parametrize("nsteps", [1, 2, 3])
@pytest.mark.parametrize("n", [11, 197])
def test_odd_and_even_steps(n, nsteps):
    """p = 6 in FP32: 242 elements, and 77,618, whose state (70 MB) is beyond the
    64 MB that get a second scratch state."""
    torch = _torch()
    s = _solver(mg.periodic_square(n, n, 10.0, 10.0), 6, 2, 1.0)
    print("[gpu-case] %d steps K=%d" % (nsteps, s.K), flush=True)
    U = _state(torch, s, 6)
    want, K1w, _ = _chain(torch, s, U, nsteps, 1e-6, (0.0, 0.0))
    got, K1 = U.clone(), torch.zeros_like(U)
    s.rk_steps(got, K1, nsteps, 1e-6)
    assert torch.equal(got, want) and torch.equal(K1, K1w)
    got, K1 = U.clone(), torch.zeros_like(U)
    for _ in range(nsteps):
        s.rk_step(got, K1, 1e-6)
    assert torch.equal(got, want) and torch.equal(K1, K1w)
    s.close()
