"""Narrow Gaussian patch masks over exactly black squares: the squares of the
masked patch fall below the normal FP64 range there, so its statistics have to
be summed in the order of the definition.  Bars: the vectors within the proven
bound, tau and masks as the oracle's."""
import numpy as np
import pytest
from test_gpu_parity import ctx  # noqa: F401
from test_gpu_patch_tiles import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,k", [(3, 50), (7, 98), (9, 60), (11, 50)])
@pytest.mark.parametrize("sigma", [0.0367, 0.05, 0.075, 0.1104, 0.184])
def test_black_squares(ctx, p, k, sigma):  # noqa: F811
    rgb = np.random.default_rng(p).random((3, 40, 66), dtype=np.float32)
    rgb.reshape(3, 40, 66)[:, (np.arange(40)[:, None] % 16 < 8) & (np.arange(66) % 16 < 8)] = 0.0
    _check(ctx, rgb, p, k, sigma, seed=3)
