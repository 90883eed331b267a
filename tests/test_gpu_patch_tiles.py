"""Patch analysis up to 11 x 11 at the sizes where its variants change: one to
four operator blocks per wave (and fewer blocks than waves), tiles of 64 pixels
with remainders, images smaller than a patch; and nearly flat patches, whose
statistics are summed entry by entry.  Bars: the vectors within the proven
bound, tau and masks as the oracle's."""
import numpy as np
import pytest
import torch
from test_gpu_parity import bound_coef, ctx, dev, masks_u64  # noqa: F401

import oracle

pytestmark = pytest.mark.gpu


def _check(ctx, rgb, p, k, sigma, seed):
    rng = np.random.default_rng(seed)
    om = rng.standard_normal((k, p * p)).astype(np.float32)
    om /= np.linalg.norm(om, axis=1, keepdims=True)
    ref = oracle.analyze(rgb, p, sigma, om)
    tau_ref, _ = oracle.tau_median(ref, 0.3)
    m_ref = oracle.cosupport(ref, tau_ref)
    rown = np.linalg.norm(om.astype(np.float64), axis=1)[None, :]
    for prec in ("fp32", "bf16"):
        a = ctx.analyze_patches(dev(rgb), p, sigma, dev(om), precision=prec)
        err = np.abs(a.cpu().numpy().astype(np.float64) - ref)
        assert np.all(err <= bound_coef(prec, p * p) * rown + 2.0 ** -100), float(err.max())
        m = ctx.cosupport(dev(rgb), p, sigma, dev(om), tau_ref, precision=prec)
        assert np.array_equal(masks_u64(m), m_ref)
        am, mm, tau = ctx.cosupport_median(dev(rgb), p, sigma, dev(om), 0.3, precision=prec)
        assert torch.equal(am, a)
        assert float(tau) == tau_ref
        assert np.array_equal(masks_u64(mm), m_ref)


@pytest.mark.parametrize("H,W,p,k", [(9, 63, 3, 16), (8, 64, 3, 32), (4, 5, 3, 33), (7, 65, 5, 64), (6, 70, 5, 65),
                                     (5, 129, 7, 130), (9, 48, 7, 17), (8, 16, 7, 256), (6, 130, 9, 200),
                                     (12, 80, 9, 128), (7, 64, 11, 256), (6, 17, 11, 1), (6, 66, 11, 193)])
def test_tiles(ctx, H, W, p, k):  # noqa: F811
    rgb = np.random.default_rng(H * W + k).random((3, H, W), dtype=np.float32)
    _check(ctx, rgb, p, k, 0.4 * p, seed=k)


@pytest.mark.parametrize("p", [3, 7, 11])
@pytest.mark.parametrize("sigma", [40.0, 4000.0])
def test_nearly_flat_patches(ctx, p, sigma):  # noqa: F811
    rng = np.random.default_rng(p)
    rgb = np.full((3, 24, 100), 0.625, np.float32)
    rgb[:, :, 30:50] += 2.0 ** -20 * rng.integers(0, 2, (3, 24, 20)).astype(np.float32)
    rgb[:, :, 50:70] += 2.0 ** -8 * rng.random((3, 24, 20), dtype=np.float32)
    rgb[:, :, 70:] = rng.random((3, 24, 30), dtype=np.float32)
    _check(ctx, rgb, p, 50, sigma, seed=3)
