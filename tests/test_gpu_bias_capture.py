"""Setting the output bias takes no memory of the context, so it can be captured
into a graph on a context that has run nothing yet; the replays follow the
rows."""
import numpy as np
import pytest
import torch
from test_gpu_mlp import dev, mlp_init

from oracle import mlp as om

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_out", [(1000, 10), (70000, 16)])
def test_output_bias_in_a_graph(n, n_out):
    from paper_1312_4746_amd import Context, Mlp
    rng = np.random.default_rng(n)
    c = Context(0)
    net = Mlp(c, 7, n_out, dev(mlp_init(7, 128, n_out, 1)))
    ell = torch.zeros((n, n_out), device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        net.fit_output_bias(ell)
    for _ in range(4):
        rows = (rng.standard_normal((n, n_out)) * 5 - 10).astype(np.float32)
        ell.copy_(torch.from_numpy(rows))
        g.replay()
        torch.cuda.synchronize()
        b3 = net.params().cpu().numpy()[-n_out:].astype(np.float64)
        ref = om.clip_targets(rows.astype(np.float64)).mean(0)
        np.testing.assert_allclose(b3, ref, rtol=2.0 ** -23, atol=0)
    net.close()
    c.close()
