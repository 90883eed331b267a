"""The co-support call on vectors long enough for a sampled bracket of the
median: every width of the mask words, a pixel count that no tile divides,
operators whose sample misses the median (rows of very different norm at a size
whose sample favours some of them), whose median is 0, or whose magnitudes leave
a gap there, and entries that are not finite.  Oracle: the separate calls, which
pass over all entries, bit for bit."""
import pytest
import torch
from test_gpu_parity import ctx, dev  # noqa: F401

pytestmark = pytest.mark.gpu


def _check(ctx, rgb, p, om, precisions=("fp32", "bf16")):
    for prec in precisions:
        a, m, tau = ctx.cosupport_median(rgb, p, 1.5, om, 0.3, precision=prec)
        a2 = ctx.analyze_patches(rgb, p, 1.5, om, precision=prec)
        assert torch.equal(a.view(torch.int32), a2.view(torch.int32))
        a2 = ctx.analyze_patches(rgb, p, 1.5, om)
        tau2 = ctx.tau_median(rgb, p, 1.5, om, a2, 0.3)
        assert float(tau) == tau2
        assert torch.equal(m, ctx.cosupport(rgb, p, 1.5, om, tau2, alpha=a2))


def _image(H, W, seed):
    g = torch.Generator().manual_seed(seed)
    return torch.rand(3, H, W, generator=g).cuda()


def _operator(k, p, seed):
    g = torch.Generator().manual_seed(seed)
    om = torch.randn(k, p * p, generator=g)
    return (om / om.norm(dim=1, keepdim=True)).cuda()


@pytest.mark.parametrize("H,W,p,k", [(900, 1001, 3, 16), (700, 705, 5, 31), (725, 727, 3, 64), (600, 601, 5, 98),
                                     (513, 515, 7, 130), (400, 447, 7, 242), (300, 287, 9, 160), (280, 321, 9, 256),
                                     (449, 451, 11, 242), (400, 401, 3, 256), (641, 643, 13, 100)])
def test_shapes(ctx, H, W, p, k):  # noqa: F811
    assert H * W * k >= 12 << 20
    _check(ctx, _image(H, W, k), p, _operator(k, p, p))


def test_sample_favours_rows(ctx):  # noqa: F811
    H, W, k = 480, 720, 172
    # rows by how often the golden ratio's multiples fall on them
    count = H * W * k
    n = torch.zeros(k, dtype=torch.int64)
    for i in range(1 << 17):
        n[((i * 0x9E3779B97F4A7C15) % (1 << 64) * count >> 64) % k] += 1
    rare = n.argsort()[: k // 2]
    assert n[rare].sum() < 0.48 * (1 << 17)
    om = _operator(k, 3, 5)
    om[rare] *= 0.25
    _check(ctx, _image(H, W, 6), 3, om)
    _check(ctx, _image(H, W, 6), 13, torch.cat([om.repeat(1, 18), om[:, :7]], 1).contiguous(), ("fp32",))


def test_ties_fill_a_list(ctx):  # noqa: F811
    # few distinct patches: one magnitude holds the median and a large share of
    # the entries, more than the places of the waves that meet them
    H, W, k = 900, 900, 17
    rgb = _image(2, 2, 12).repeat(1, H // 2, W // 2).contiguous()
    om = _operator(1, 3, 13).repeat(k, 1).contiguous()
    _check(ctx, rgb, 3, om)


def test_median_zero_and_gap(ctx):  # noqa: F811
    om = _operator(128, 3, 7)
    rgb = _image(600, 500, 8)
    rgb[:, :, :300] = 0.5
    rgb[:, :, :300] *= 0.0
    _check(ctx, rgb, 3, om)
    om2 = om.clone()
    om2[::2] *= 2.0 ** -12
    _check(ctx, _image(600, 500, 9), 3, om2)


def test_not_finite(ctx):  # noqa: F811
    om = _operator(128, 3, 10)
    om[5] *= 3.0e38  # sums overflow
    _check(ctx, _image(600, 500, 11), 3, om)
