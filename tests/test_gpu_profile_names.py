"""Timing spans: every step's name records, also where one launch does the work
of several, and the analysis' span holds its kernel alone."""
import pytest
import torch
from test_gpu_parity import ctx, dev  # noqa: F401

from workloads import make_workload

pytestmark = pytest.mark.gpu


def _counts(ctx, call, names):  # noqa: F811
    call()
    ctx.profile_enable(True)
    call()
    got = {n: ctx.profile_read(n) for n in names}
    ctx.profile_enable(False)
    for n in names:  # a name of a shared launch can be recorded on its own
        ctx.profile_only(n)
        ctx.profile_enable(True)
        call()
        ms, cnt = ctx.profile_read(n)
        assert cnt == got[n][1] and (ms > 0) == (cnt > 0), n
        ctx.profile_enable(False)
    ctx.profile_only(None)
    return {n: c for n, (_, c) in got.items()}


def test_clustering(ctx):  # noqa: F811
    from paper_1312_4746_amd import UnsupParams
    rgb = torch.rand(3, 20, 30, device="cuda")
    masks = torch.zeros((600, 1), dtype=torch.int64, device="cuda")
    prm = UnsupParams(colour_classes=2, texture_classes=2, iterations=2)
    got = _counts(ctx, lambda: ctx.unsupervised_loglik(rgb, masks, 8, [0, 1], [2, 3], prm), ["kmeans", "kmedians"])
    assert got == {"kmeans": 1, "kmedians": 1}


def test_training(ctx):  # noqa: F811
    from paper_1312_4746_amd import Mlp, param_count
    net = Mlp(ctx, 9, 3, torch.randn(param_count(9, 128, 3), device="cuda") * 0.1)
    x, ell = torch.randn(32, 9, device="cuda"), torch.randn(32, 3, device="cuda")
    order = torch.arange(32, dtype=torch.int32, device="cuda").repeat(3)
    names = ["mlp_fwdbwd", "mlp_wgrad", "mlp_adam"]
    assert _counts(ctx, lambda: net.train(x, ell, order, 32), names) == dict.fromkeys(names, 3)
    net.close()


@pytest.mark.parametrize("W", [40, 2100])  # the matrix-core path and the exact one
def test_data_term(ctx, W):  # noqa: F811
    w = make_workload("prof", H=24, W=W, R=2, p=3, k=20, seed=1, per_region=6)
    masks = torch.zeros((w.N, 1), dtype=torch.int64, device="cuda")
    args = (dev(w.rgb), masks, w.k, dev(w.sample_pix), dev(w.sample_label), w.L)
    got = _counts(ctx, lambda: ctx.label_loglik(*args), ["coef", "stream", "parzen"])
    assert got == {"coef": 1, "stream": int(W <= 2048), "parzen": 1}


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_analysis_within_the_median(ctx, prec):  # noqa: F811
    H, W, p, k = 600, 601, 5, 98
    rgb = torch.rand(3, H, W, device="cuda")
    om = torch.randn(k, p * p, device="cuda")
    got = _counts(ctx, lambda: ctx.cosupport_median(rgb, p, 1.5, om, 0.3, precision=prec), ["analyze", "analyze_bf16"])
    assert got == {"analyze": 1, "analyze_bf16": int(prec == "bf16")}
    ctx.profile_enable(True)
    for _ in range(5):
        ctx.cosupport_median(rgb, p, 1.5, om, 0.3, precision=prec)
    ms, names = {}, ["analyze", "tau_select", "cosupport"]
    for n in names:
        ms[n] = ctx.profile_read(n)
    ctx.profile_enable(False)
    # the bracket's steps before and after the analysis have spans of their own
    assert ms["tau_select"][1] == 10 and ms["cosupport"][1] == 10, ms
