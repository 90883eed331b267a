"""The exact median where one value, or a few, or a cluster far narrower than the
candidate window, is held by a large share of the entries: flat images, repeated
patterns with and without noise of one unit in the last place, black areas (zero
patches) up to most of the image, few grey levels.  Oracle: FP64, tau and masks
bit for bit."""
import numpy as np
import pytest
from test_gpu_parity import ctx  # noqa: F401
from test_gpu_patch_tiles import _check

pytestmark = pytest.mark.gpu


def _image(kind, H, W, rng):
    r = rng.random((3, H, W), dtype=np.float32)
    if kind == "flat":
        r[:] = 0.5
    elif kind == "dots":
        r = np.tile(r[:, :2, :2], (1, H // 2, W // 2))
    elif kind == "noisy":
        r = np.tile(r[:, :2, :2], (1, H // 2, W // 2)) * (1 + 2.0 ** -23 * rng.integers(0, 3, (3, H, W)))
    elif kind == "black":
        r[:, :, : W * 6 // 10] = 0
    elif kind == "dark":
        r[:, :, : W * 3 // 10] = 0
    elif kind == "levels":
        r = np.floor(r * 4) / 4
    return np.ascontiguousarray(r, dtype=np.float32)


@pytest.mark.parametrize("kind", ["flat", "dots", "noisy", "black", "dark", "levels"])
@pytest.mark.parametrize("H,W,p,k", [(16, 16, 3, 8), (64, 64, 5, 50), (64, 64, 3, 20), (40, 66, 7, 98), (36, 50, 11, 242),
                                     (30, 34, 15, 120)])
def test_tied_values(ctx, kind, H, W, p, k):  # noqa: F811
    _check(ctx, _image(kind, H, W, np.random.default_rng(H + p)), p, k, 0.4 * p, seed=k)


@pytest.mark.parametrize("kind", ["flat", "dots", "noisy", "black", "levels"])
def test_tied_values_long(ctx, kind):  # noqa: F811
    _check(ctx, _image(kind, 360, 380, np.random.default_rng(4)), 7, 98, 2.8, seed=5)
