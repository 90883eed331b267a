"""Calls long enough for a sampled bracket of the median against the FP64 oracle,
which shares none of the analysis: the vectors within the proven bound, tau and
masks bit for bit, where the bracket is decided inside the analysis (up to 9 x 9)
and in a pass of its own, in both precisions, with wide and narrow patch masks."""
import numpy as np
import pytest
from test_gpu_parity import ctx  # noqa: F401
from test_gpu_patch_tiles import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,p,k,sigma", [(221, 230, 3, 256, 1.1), (329, 391, 7, 98, 2.6), (329, 391, 7, 98, 0.1104),
                                           (221, 230, 9, 250, 3.0), (221, 230, 11, 250, 0.184),
                                           (221, 230, 13, 250, 4.0)])
def test_long_calls(ctx, H, W, p, k, sigma):  # noqa: F811
    assert H * W * k >= 12 << 20
    rng = np.random.default_rng(p)
    rgb = rng.random((3, H, W), dtype=np.float32)
    rgb[:, (np.arange(H)[:, None] % 48 < 8) & (np.arange(W) % 48 < 8)] = 0.0
    _check(ctx, rgb, p, k, sigma, seed=p)
