"""GPU tests of the fused training kernel at the edges of its blocks: a batch
that leaves a wave's second tile, a tile or all but one sample empty, one and
several blocks per workgroup, and both output widths at their limits."""
import numpy as np
import pytest

from oracle import closure as OC
from tests.test_gpu_closure import _net_case, _oracle_inputs, _rel, _say, _torch, _unpack

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_out,B", [(24, 1), (32, 64), (1, 65), (24, 16384), (32, 16385), (24, 20001), (17, 49217),
                                     (33, 1), (64, 65), (60, 16449)])
def test_fused_training_block_edges(n_out, B):
    """Up to 16,384 samples a workgroup has one 64-sample block (one tile a
    wave), beyond it whole 128-sample blocks, the last perhaps half empty.  The
    gradient is within the network's bound (3e-2 normwise) of the FP64 oracle,
    the loss, a square, within twice the forward bound, and both are
    reproducible."""
    torch = _torch()
    from paper_2508_17917_amd import _lib as L
    params, X, T, norm = _net_case(7, B=B, n_out=n_out)
    q, Xn, Tn = _oracle_inputs(params, X, T, norm, n_out=n_out)
    lo, go = OC.loss_and_grads(q, Xn, Tn)
    Xd, Td = torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda()
    m = L.dg_mlp_create(28, 128, n_out, B)
    L.dg_mlp_set_params(m, params)
    L.dg_mlp_set_normalization(m, *norm)
    _say("fused training n_out=%d B=%d" % (n_out, B))
    loss = L.dg_mlp_backward(m, Xd, Td)
    g = L.dg_mlp_get_grad(m)
    assert L.dg_mlp_backward(m, Xd, Td) == loss
    assert np.array_equal(g, L.dg_mlp_get_grad(m)), "not reproducible"
    L.dg_mlp_destroy(m)
    assert abs(loss - lo) <= 3e-2 * lo
    got = _unpack(g, n_out=n_out)
    for k in go:
        assert _rel(got[k], go[k]) <= 3e-2, k


@pytest.mark.parametrize("n_out,B", [(24, 16385), (32, 20001), (17, 49217), (24, 65), (17, 97), (60, 16449)])
def test_fused_training_last_block_decides(n_out, B):
    """The samples of the last, partly filled block carry nearly all of the loss
    and gradient (their targets are ten thousand standard deviations off, the
    others' one): a sample of it left out, or a row past the end counted, is far
    outside the bounds, which are those of a batch of one."""
    torch = _torch()
    from paper_2508_17917_amd import _lib as L
    params, X, T, norm = _net_case(7, B=B, n_out=n_out)
    tail = (B - 1) % 64 + 1
    rng = np.random.default_rng(B)
    T[-tail:] = norm[2] + 1e4 * norm[3] * rng.standard_normal((tail, n_out)).astype(T.dtype)
    q, Xn, Tn = _oracle_inputs(params, X, T, norm, n_out=n_out)
    lo, go = OC.loss_and_grads(q, Xn, Tn)
    rest, _ = OC.loss_and_grads(q, Xn[:-tail], Tn[:-tail])
    assert rest * (B - tail) < 0.05 * lo * B   # (what the case is for)
    m = L.dg_mlp_create(28, 128, n_out, B)
    L.dg_mlp_set_params(m, params)
    L.dg_mlp_set_normalization(m, *norm)
    _say("fused training tail n_out=%d B=%d" % (n_out, B))
    loss = L.dg_mlp_backward(m, torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda())
    got = _unpack(L.dg_mlp_get_grad(m), n_out=n_out)
    L.dg_mlp_destroy(m)
    assert abs(loss - lo) <= 3e-2 * lo
    for k in go:
        assert _rel(got[k], go[k]) <= 3e-2, k
