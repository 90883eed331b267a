"""The training launches at the edges of their blocks: odd and even counts of
16-feature input blocks, 1 to 16 outputs, one tile, chunk counts that are not
16 (a chain longer than the 16 tiles a wave requests at once) and the largest
batch; the inference kernel stages the same weight copies.  Bars as in
test_gpu_mlp."""
import numpy as np
import pytest
from test_gpu_mlp import _net, ctx, dev, grad_error_bound  # noqa: F401

from oracle import mlp as om

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_in,n_out,n", [(1, 1, 16), (5, 16, 48), (16, 3, 272), (17, 4, 16 * 34), (33, 16, 1024),
                                          (64, 2, 16 * 23), (97, 7, 16 * 15), (112, 10, 4096), (128, 16, 8192)])
def test_gradient_and_forward(ctx, n_in, n_out, n):  # noqa: F811
    net, p0 = _net(ctx, n_in, n_out, seed=5)
    sh = om.Shapes(n_in, 128, n_out)
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, n_in)).astype(np.float32) * 0.5
    ell = (rng.standard_normal((n, n_out)) * 5 - 10).astype(np.float32)
    g, _ = net.grad(dev(X), dev(ell))
    T = om.clip_targets(ell.astype(np.float64))
    _, g_ref = om.loss_and_grad(p0, sh, X, T, emulate_bf16=True)
    err = np.abs(g.cpu().numpy().astype(np.float64) - g_ref)
    assert np.all(err <= grad_error_bound(p0, sh, X, T)), float(err.max())
    y = net.forward(dev(X[:100])).cpu().numpy().astype(np.float64)
    ref = om.forward(p0, sh, X[:100], emulate_bf16=True)["y"]
    assert np.max(np.abs(y - ref)) <= 2e-3 * max(1.0, float(np.abs(ref).max()))
    net.fit_output_bias(dev(ell))
    b3 = net.params().cpu().numpy()[-n_out:].astype(np.float64)
    np.testing.assert_allclose(b3, T.mean(0), rtol=2.0 ** -23, atol=0)
    net.close()
