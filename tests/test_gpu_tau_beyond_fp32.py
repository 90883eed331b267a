"""Factors of the median that put tau past the FP32 range: every entry is in,
the places past k stay clear, and nothing is written past the masks or listed
past the vectors.  The general pass over the entries and both forms of the
sampled bracket (inside the analysis, and a pass of its own)."""
import pytest
import torch
from test_gpu_parity import ctx  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,p,k", [(40, 67, 7, 98), (37, 65, 11, 65), (720, 727, 3, 33), (480, 721, 11, 65)])
@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("frac", [1e38, 2e39, 1e300])
def test_every_entry_is_in(ctx, H, W, p, k, prec, frac):  # noqa: F811
    g = torch.Generator().manual_seed(k)
    rgb = torch.rand(3, H, W, generator=g).cuda()
    om = torch.randn(k, p * p, generator=g)
    om = (om / om.norm(dim=1, keepdim=True)).cuda()
    nw = (k + 63) // 64
    room = torch.zeros((H * W + 64, nw), dtype=torch.int64, device="cuda")
    a, m, tau = ctx.cosupport_median(rgb, p, 1.5, om, frac, precision=prec, out=room[32:32 + H * W])
    assert not bool(room[:32].any()) and not bool(room[32 + H * W:].any())
    med = ctx.tau_median(rgb, p, 1.5, om, ctx.analyze_patches(rgb, p, 1.5, om), 1.0)
    assert float(tau) == frac * med
    want = torch.full((nw,), -1, dtype=torch.int64)
    if k % 64:
        want[-1] = (1 << (k % 64)) - 1
    if frac > 1e38:  # (at 1e38 tau lies within the range of the entries' bounds or above)
        assert torch.equal(m, want.cuda().expand_as(m))
    assert not bool((m[:, -1] & ~want[-1].cuda()).any())
