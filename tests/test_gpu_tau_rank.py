"""The exact median of stored vectors (its candidates ranked, or selected by digits)
against the one call, whose candidates are binned: the same tau bit for bit, from
few to thousands of candidates and with one value held by very many."""
import pytest
import torch
from test_gpu_parity import ctx  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,p,k,tie", [(64, 64, 5, 50, False), (400, 500, 3, 16, False), (512, 512, 5, 50, False),
                                         (321, 481, 7, 98, False), (400, 500, 3, 16, True)])
def test_tau_of_both_calls(ctx, H, W, p, k, tie):  # noqa: F811
    g = torch.Generator().manual_seed(H)
    rgb = torch.rand(3, H, W, generator=g).cuda()
    if tie:  # a few distinct patches
        rgb = rgb[:, :4, :4].repeat(1, H // 4, W // 4).contiguous()
    om = torch.randn(k, p * p, generator=g)
    om = (om / om.norm(dim=1, keepdim=True)).cuda()
    a, _, tau = ctx.cosupport_median(rgb, p, 1.5, om, 0.3)
    assert ctx.tau_median(rgb, p, 1.5, om, a, 0.3) == float(tau)
