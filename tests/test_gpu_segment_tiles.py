"""The on-chip forms of the FP32 primal-dual iteration at the edges of their
tiles: the resident form (one launch, tiles of 30 x (rows - 2) pixels that
exchange their borders) and the tile form (several iterations a launch) that
images beyond the chip take.  Bars as in test_gpu_segment."""
import pytest
from test_gpu_segment import _check, _synthetic_term, ctx  # noqa: F401

from workloads import make_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,L,nu,iters", [
    (30, 30, 2, 0.0, 1), (31, 61, 12, 0.0, 9), (59, 91, 13, 7.0, 6), (200, 33, 16, 30.0, 5), (5, 900, 6, 3.0, 4),
    (25, 40, 1, 2.0, 3), (90, 151, 16, 0.0, 40), (91, 30, 5, 9.0, 40), (321, 481, 16, 50.0, 12),
    # more tiles than compute units
    (430, 411, 13, 0.0, 7), (430, 411, 13, 30.0, 3), (521, 530, 4, 0.0, 10), (521, 530, 2, 8.0, 5)])
def test_tile_edges(ctx, H, W, L, nu, iters):  # noqa: F811
    w = make_workload("seg_tiles", H=H, W=W, R=max(2, min(L, 6)), p=3, k=8, seed=17, per_region=1)
    w.L = L
    w.region = w.region % L
    _check(ctx, w.rgb, _synthetic_term(w, seed=L), 1.5, nu, iters, "fp32")


def test_radii_beyond_the_short_root_and_quotient(ctx):  # noqa: F811
    """lambda = 0 (radius 0) and a small gamma (radii down to 0 at strong
    edges) take the full square root and quotient."""
    w = make_workload("seg_tiles", H=45, W=70, R=3, p=3, k=8, seed=18, per_region=1)
    ll = _synthetic_term(w, seed=5)
    for lam in (0.0, 1e-12, 2.0):
        _check(ctx, w.rgb, ll, lam, 0.0, 20, "fp32")
    w.rgb[:, :, 35:] *= 0.01
    _check(ctx, w.rgb, ll, 1.0, 0.0, 20, "fp32")


@pytest.mark.parametrize("H,W,L,nu,prec", [(23, 29, 64, 0.0, "fp32"), (33, 40, 63, 4.0, "fp64"), (16, 16, 33, 2.0, "fp32"),
                                           (257, 3, 16, 5.0, "fp32")])
def test_start_and_finish_at_the_label_limits(ctx, H, W, L, nu, prec):  # noqa: F811
    """The planes turned in LDS (up to 64 labels x 256 pixels) and the energies'
    rows, partial last workgroups among them."""
    w = make_workload("seg_tiles", H=H, W=W, R=2, p=3, k=8, seed=19, per_region=1)
    w.L = L
    w.region = w.region % L
    for iters in (0, 2):
        _check(ctx, w.rgb, _synthetic_term(w, seed=L), 1.0, nu, iters, prec)
