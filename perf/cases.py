"""Workloads of the co-sparse segmentation library, each through its public
Python entry points: the co-support front end, the per-label data term in its
forms, whole images, the segmentation by convex relaxation, the unsupervised
mode, and the learned surrogate's training and inference.

Sizes are those of the paper's experiments and of this repository's benchmark
(64 x 64, the 481 x 321 images of BSDS, 1024 x 1024, 2048 x 2048), with odd
sizes between them.  Inputs are synthetic: Voronoi regions with their own mean
colour and oriented texture, painted with 13-pixel brush strokes, drawn on the
GPU from the seed alone.  `exact` evaluates each path from its definition in
64 bits with plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1312_4746_amd import Context, LoglikParams, Mlp, SegmentParams, UnsupParams

HID = 128
CLIP = 20.0
SIGMA_IOTA = 0.01  # the paper's smooth co-support map
TAU_FRAC = 0.1

_BASE = dict(p=7, k=98, L=10, M=0, levels=255, precision="fp32", form="sum", normalise=False, subset=0,
             iters=0, nu=0.0, batch=0, steps=0)


def _case(kind, H, W, **kw):
    return dict(_BASE, kind=kind, H=H, W=W, **kw)


def listed():
    return [
        # one interactive refresh of a small image (or a crop of one): latency
        dict(_case("image", 64, 64, p=5, k=50, L=3, M=600), name="image_64"),
        # one benchmark image, from pixels to the data term of every label
        dict(_case("image", 321, 481, M=7720), name="image_bsds"),
        # co-supports of a large image with the largest operator in use
        dict(_case("front", 1024, 1024, p=11, k=242), name="front_1024"),
        # co-supports of a frame in the BF16 form that feeds the surrogate
        dict(_case("front", 2048, 2048, precision="bf16"), name="front_2048_bf16"),
        # the data term of a large image with many labels: the headline workload
        dict(_case("loglik", 1024, 1024, p=11, k=242, L=16, M=50000), name="loglik_1024"),
        # an odd-sized image whose colours are plain floats, labels normalised
        dict(_case("loglik", 389, 517, L=7, M=9001, levels=0, normalise=True), name="loglik_float_odd"),
        # the paper's own setting: smooth co-supports, median representatives
        dict(_case("loglik", 321, 481, M=7720, form="soft"), name="soft_bsds"),
        # exact targets at the surrogate's training pixels (2 % of a frame)
        dict(_case("loglik", 2048, 2048, M=209715, subset=83886), name="targets_2048"),
        # the segmentation of one benchmark image
        dict(_case("segment", 321, 481, iters=300), name="segment_bsds"),
        # unsupervised segmentation of one benchmark image (16 classes, label cost)
        dict(_case("unsup", 321, 481, L=16, iters=300, nu=1100.0), name="unsup_bsds"),
        # fitting the surrogate of one image
        dict(_case("fit", 1024, 1024, M=20000, batch=4096, steps=100), name="fit_4096"),
        # one frame by the trained surrogate, unsure pixels by the exact data term
        dict(_case("fallback", 2048, 2048, M=209715), name="fallback_2048"),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _image_size(rng, lo, hi):
    n = _log(rng, lo, hi)
    a = _log(rng, 0.5, 2.0)
    H = max(32, int(math.sqrt(n * a)))
    return H, max(32, int(n / H))


def draw(rng):
    kind = rng.choice(["image", "image", "front", "front", "loglik", "loglik", "loglik", "list", "segment", "unsup",
                       "fit", "infer", "fallback"])
    p = rng.choice([5, 7, 7, 9, 11])
    k = min(256, rng.randint(p * p, 2 * p * p + 1))
    L = rng.randint(2, 16)
    precision = rng.choice(["fp32", "fp32", "bf16"])
    if kind == "front":
        H, W = _image_size(rng, 4096, min(2.0 ** 22, 4.0e8 / k, 3.0e10 / (k * p * p)))
        return _case("front", H, W, p=p, k=k, precision=precision)
    if kind in ("image", "loglik"):
        H, W = _image_size(rng, 4096, 2.0 ** 20)
        M = int(min(H * W * _log(rng, 0.01, 0.15), 5.0e10 / (H * W)))
        levels = rng.choice([255, 255, 0])
        if levels == 0:  # the colour term of plain floats costs more
            M = min(M, int(2.0e10 / (H * W)))
        M = max(M, 16 * L)
        form = rng.choice(["sum", "sum", "joint", "soft"]) if kind == "loglik" else "sum"
        return _case(kind, H, W, p=p, k=k, L=L, M=M, levels=levels, form=form, normalise=rng.random() < 0.3,
                     precision=precision if kind == "image" else "fp32")
    if kind == "list":
        H, W = _image_size(rng, 2.0 ** 16, 2.0 ** 22)
        M = int(H * W * _log(rng, 0.01, 0.05))
        return _case("loglik", H, W, p=7, k=rng.randint(49, 99), L=L, M=M, levels=rng.choice([255, 0]),
                     subset=int(_log(rng, 64, 0.02 * H * W)))
    if kind == "segment":
        iters = rng.choice([50, 100, 200, 300])
        H, W = _image_size(rng, 4096, min(2.0 ** 20, 2.0e9 / (iters * L)))
        return _case("segment", H, W, L=L, iters=iters, nu=rng.choice([0.0, 0.0, 50.0]),
                     precision=rng.choice(["fp32", "fp32", "fp32", "fp64"]))
    if kind == "unsup":
        L = rng.choice([4, 9, 16])
        H, W = _image_size(rng, 4096, 2.0 ** 18)
        return _case("unsup", H, W, p=p, k=k, L=L, iters=rng.choice([100, 300]), nu=rng.choice([300.0, 1100.0]))
    k = rng.randint(40, 123)
    L = rng.randint(2, 16)
    if kind == "fit":
        H, W = _image_size(rng, 2.0 ** 14, 2.0 ** 20)
        return _case("fit", H, W, k=k, L=L, M=max(32 * L, H * W // 50), batch=16 * int(_log(rng, 16, 512)),
                     steps=rng.randint(20, 100))
    H, W = _image_size(rng, 2.0 ** 14, 2.0 ** 22)
    return _case(kind, H, W, k=k, L=L, M=max(32 * L, H * W // 20))


# ---- inputs -----------------------------------------------------------------
_CTX = []


def _context():
    """The process's one library context, kept as a user's program keeps it."""
    if not _CTX:
        _CTX.append(Context(torch.cuda.current_device()))
    return _CTX[0]


def _gen(seed, part):
    return torch.Generator(device="cuda").manual_seed(1000003 * int(seed) + part)


def _scene(case, seed):
    """(region (N,), rgb (3, H, W) float32): Voronoi regions, one oriented
    sinusoid each, noise; with levels n > 0 stored at n levels per channel."""
    H, W, L = case["H"], case["W"], case["L"]
    for attempt in range(64):
        g = _gen(seed, 17 * attempt)
        c = torch.rand(L, 2, generator=g, device="cuda", dtype=torch.float64)
        yy = torch.arange(H, device="cuda", dtype=torch.float64)[:, None]
        xx = torch.arange(W, device="cuda", dtype=torch.float64)[None, :]
        best = torch.full((H, W), math.inf, device="cuda", dtype=torch.float64)
        region = torch.zeros((H, W), device="cuda", dtype=torch.int64)
        for r in range(L):
            d = (xx - c[r, 0] * W) ** 2 + (yy - c[r, 1] * H) ** 2
            upd = d < best
            best = torch.where(upd, d, best)
            region = torch.where(upd, r, region)
        if int(torch.bincount(region.flatten(), minlength=L).min()) * 6 * L >= H * W:
            break
    prm = torch.rand(6, L, generator=g, device="cuda", dtype=torch.float64)
    period, theta, phase = 3.0 + 9.0 * prm[3], math.pi * prm[4], 2.0 * math.pi * prm[5]
    tex = 0.1 * torch.sin(2.0 * math.pi * (xx * torch.cos(theta)[region] + yy * torch.sin(theta)[region])
                          / period[region] + phase[region])
    rgb = torch.stack([prm[ch][region] + tex for ch in range(3)])
    rgb = (rgb + 0.05 * torch.randn(3, H, W, generator=g, device="cuda", dtype=torch.float64)).clamp(0.0, 1.0)
    if case["levels"]:
        rgb = torch.round(rgb * case["levels"]) / case["levels"]
    return region.flatten(), rgb.float().contiguous()


def _scribbles(case, region, seed):
    """(pixels, labels) int32: random-walk strokes of a 13-pixel brush inside
    each region, shares in proportion to the regions' areas, in painting order."""
    H, W, L, M = case["H"], case["W"], case["L"], case["M"]
    N = H * W
    g = _gen(seed, 5)
    area = torch.bincount(region, minlength=L).cpu().numpy()
    want = np.maximum(1, np.floor(M * area / N)).astype(np.int64)
    want = np.minimum(want, area)
    i = 0
    while want.sum() != M and i < 64 * L:  # the shares add up to M
        r, i = i % L, i + 1
        step = int(np.clip(M - want.sum(), 1 - want[r], area[r] - want[r]))
        want[r] += step
    walks = [int(math.ceil(t / 250)) + 1 for t in want]
    owner = torch.repeat_interleave(torch.arange(L, device="cuda"), torch.tensor(walks, device="cuda"))
    by_region = torch.argsort(region, stable=True)
    first = torch.tensor(np.concatenate([[0], np.cumsum(area)[:-1]]), device="cuda")
    areas = torch.tensor(area, device="cuda")
    nw, steps = owner.numel(), 200
    pick = (torch.rand(nw, generator=g, device="cuda", dtype=torch.float64) * areas[owner]).long()
    start = by_region[first[owner] + torch.minimum(pick, areas[owner] - 1)]
    turn = torch.rand(nw, steps, generator=g, device="cuda") >= 0.7
    turn[:, 0] = True
    d = torch.randint(0, 8, (nw, steps), generator=g, device="cuda")
    last = torch.cummax(torch.where(turn, torch.arange(steps, device="cuda")[None, :], 0), dim=1).values
    d = torch.gather(d, 1, last)
    dirs = torch.tensor([(1, 0), (1, 1), (0, 1), (-1, 1), (-1, 0), (-1, -1), (0, -1), (1, -1)], device="cuda")
    path = torch.cumsum(dirs[d], dim=1)
    off = [(u, v) for v in range(-6, 7) for u in range(-6, 7) if u * u + v * v <= 6.5 ** 2]
    key = torch.full((N,), nw * steps, device="cuda", dtype=torch.int64)
    stamp = torch.arange(nw * steps, device="cuda").reshape(nw, steps)
    for u, v in off:
        x, y = (start % W)[:, None] + path[..., 0] + u, (start // W)[:, None] + path[..., 1] + v
        lin = y.clamp(0, H - 1) * W + x.clamp(0, W - 1)
        ok = (x >= 0) & (x < W) & (y >= 0) & (y < H)
        ok &= region[lin] == owner[:, None]
        key.scatter_reduce_(0, torch.where(ok, lin, 0).flatten(),
                            torch.where(ok, stamp, nw * steps).flatten(), "amin")
    order = torch.argsort(region * (nw * steps + 1) + key, stable=True)
    pix = torch.cat([order[int(first[r]):int(first[r]) + int(want[r])] for r in range(L)])
    lab = torch.repeat_interleave(torch.arange(L, device="cuda"), torch.tensor(want, device="cuda"))
    return pix.int().contiguous(), lab.int().contiguous()


def _operator(case, seed):
    g = _gen(seed, 7)
    om = torch.randn(case["k"], case["p"] ** 2, generator=g, device="cuda", dtype=torch.float64)
    om = om - om.mean(1, keepdim=True)
    return (om / om.norm(dim=1, keepdim=True)).float().contiguous()


def _reflect(n, h):
    i = torch.arange(-h, n + h, device="cuda")
    i = torch.where(i < 0, -i - 1, i)
    return torch.where(i >= n, 2 * n - i - 1, i)


def _analysed(case, rgb, om, dtype):
    """Analysed vectors of every pixel from the definition, in 64 bits, kept as `dtype`."""
    H, W, p, k = case["H"], case["W"], case["p"], case["k"]
    h = p // 2
    r = rgb.double()
    gray = (0.299 * r[0] + 0.587 * r[1]) + 0.114 * r[2]
    pad = gray[_reflect(H, h)][:, _reflect(W, h)]
    e = torch.arange(-h, h + 1, device="cuda", dtype=torch.float64)
    w = torch.exp(-(e[:, None] ** 2 + e[None, :] ** 2) / (2.0 * (p / 4.0) ** 2)).flatten()
    omt = om.double().t().contiguous()
    out = torch.empty(H * W, k, device="cuda", dtype=dtype)
    rows = max(1, (1 << 19) // W)
    for y in range(0, H, rows):
        n = min(rows, H - y)
        s = pad[y:y + n + 2 * h].unfold(0, p, 1).unfold(1, p, 1).reshape(n * W, p * p) * w
        s = s - s.mean(1, keepdim=True)
        nu = s.norm(dim=1, keepdim=True)
        s = torch.where(nu > 0, s / nu, torch.zeros_like(s))
        out[y * W:(y + n) * W] = (s @ omt).to(dtype)
    return out


def _masks(alpha, frac=TAU_FRAC):
    """Co-support words (N, ceil(k/64)) int64 at about the given share of the median."""
    N, k = alpha.shape
    a = alpha.flatten()
    tau = frac * a[:: max(1, a.numel() // 1000003)].abs().median()
    words = torch.zeros(N, (k + 63) // 64, device="cuda", dtype=torch.int64)
    for j in range(k):
        words[:, j // 64] |= (alpha[:, j].abs() <= tau).long() << (j % 64)
    return words


def _bits(words, k):
    j = torch.arange(k, device="cuda")
    return ((words[:, j // 64] >> (j % 64)) & 1).float()


def _params(case):
    return LoglikParams(normalise=case["normalise"], colour_levels=case["levels"])


def _rows(case, rgb, alpha, pix):
    """Surrogate input rows of the listed pixels."""
    H, W = case["H"], case["W"]
    pos = torch.stack([(pix % W).float() / max(W - 1, 1), (pix // W).float() / max(H - 1, 1)], 1)
    return torch.cat([rgb.reshape(3, -1)[:, pix].t(), pos, alpha[pix]], 1).contiguous()


def _net_init(case, seed):
    g = _gen(seed, 11)
    parts = []
    for out, fan in ((HID, 5 + case["k"]), (HID, HID), (case["L"], HID)):
        b = 1.0 / math.sqrt(fan)
        parts += [(2.0 * torch.rand(out * fan, generator=g, device="cuda", dtype=torch.float64) - 1.0) * b,
                  (2.0 * torch.rand(out, generator=g, device="cuda", dtype=torch.float64) - 1.0) * b]
    return torch.cat(parts)


def _net_split(flat, k, L):
    n, at, out = 5 + k, 0, []
    for shape in ((HID, n), (HID,), (HID, HID), (HID,), (L, HID), (L,)):
        m = int(np.prod(shape))
        out.append(flat[at:at + m].reshape(shape))
        at += m
    return out


def _gelu(z):
    return z * 0.5 * (1.0 + torch.erf(z / math.sqrt(2.0)))


def _net_hidden(ps, x):
    return _gelu(_gelu(x @ ps[0].t() + ps[1]) @ ps[2].t() + ps[3])


def _net_trained(case, seed, x, ell):
    """A network of the trained ones' behaviour, without the library: seeded
    hidden layers with wide first weights, the last layer fitted to the clipped
    targets by least squares in 64 bits."""
    k, L = case["k"], case["L"]
    flat = _net_init(case, seed)
    ps = _net_split(flat, k, L)
    ps[0][:, :5] *= 12.0
    ps[0][:, 5:] *= 3.0
    ps[2].mul_(3.0)
    t = torch.maximum(ell, ell.max(1, keepdim=True).values - CLIP)
    h = torch.cat([_net_hidden(ps, x.double()), torch.ones(x.shape[0], 1, device="cuda", dtype=torch.float64)], 1)
    a = (h.t() @ h).cpu() + 1e-3 * torch.eye(HID + 1, dtype=torch.float64)
    sol = torch.linalg.solve(a, (h.t() @ t).cpu()).to("cuda")
    ps[4].copy_(sol[:HID].t())
    ps[5].copy_(sol[HID])
    return flat.float().contiguous()


def _data_terms(case, region, seed):
    """Log-likelihoods of the kind the convex relaxation gets: high at a
    pixel's own region, noisy, lower elsewhere."""
    N, L = region.numel(), case["L"]
    g = _gen(seed, 13)
    ll = -8.0 + 2.5 * torch.randn(N, L, generator=g, device="cuda")
    ll[torch.arange(N, device="cuda"), region] += 5.0
    return ll.contiguous()


def _classes(case):
    return int(round(math.sqrt(case["L"])))


def _inputs(case, seed):
    """Every input of the case, on the GPU, without the library."""
    s = {}
    region, s["rgb"] = _scene(case, seed)
    kind, N = case["kind"], case["H"] * case["W"]
    if kind == "segment":
        s["ll"] = _data_terms(case, region, seed)
        return s
    s["om"] = _operator(case, seed)
    if case["M"]:
        s["pix"], s["lab"] = _scribbles(case, region, seed)
    if kind in ("front", "image"):
        return s
    alpha = _analysed(case, s["rgb"], s["om"], torch.float32)
    if kind == "loglik" and case["form"] == "soft":
        s["alpha"] = alpha
        return s
    s["masks"] = _masks(alpha)
    if kind == "unsup":
        init = torch.randperm(N, generator=_gen(seed, 19), device="cuda")[:2 * _classes(case)].cpu().numpy()
        s["init"] = (init[:_classes(case)], init[_classes(case):])
    if case["subset"]:
        s["subset"] = torch.randperm(N, generator=_gen(seed, 23), device="cuda")[:case["subset"]].sort().values.int()
    if kind in ("fit", "infer", "fallback"):
        rows = max(2 * case["batch"], 4096) if kind == "fit" else 4096
        tp = torch.randperm(N, generator=_gen(seed, 29), device="cuda")[:rows].sort().values
        ell = _loglik64(dict(case, form="sum", normalise=False), s, tp)
        x = _rows(case, s["rgb"], alpha, tp)
        if kind == "fit":
            s["x"], s["ell"] = x, ell.float().contiguous()
            need, got = case["batch"] * case["steps"], []
            g = _gen(seed, 31)
            while sum(t.numel() for t in got) < need:
                got.append(torch.randperm(x.shape[0], generator=g, device="cuda"))
            s["order"] = torch.cat(got)[:need].int().contiguous()
            s["net"] = _net_init(case, seed).float().contiguous()
        else:
            s["alpha"] = alpha
            s["net"] = _net_trained(case, seed, x, ell)
    return s


def prepare(case, seed):
    """The inputs, the process's context, the output buffers that a program
    working through images of one size keeps, and the trained network."""
    s = _inputs(case, seed)
    s["case"], s["ctx"] = case, _context()
    N, k, L, kind = case["H"] * case["W"], case["k"], case["L"], case["kind"]
    if kind in ("front", "image"):
        s["alpha"] = torch.empty(N, k, device="cuda")
        s["masks"] = torch.empty(N, (k + 63) // 64, device="cuda", dtype=torch.int64)
        s["tau"] = torch.empty(1, device="cuda", dtype=torch.float64)
    if kind in ("image", "loglik"):
        s["out"] = torch.empty(case["subset"] or N, L, device="cuda")
    if kind in ("infer", "fallback"):
        s["mlp"] = Mlp(s["ctx"], 5 + k, L, s["net"])
        s["out"] = torch.empty(N, L, device="cuda")
    return s


def run(s):
    case, ctx = s["case"], s["ctx"]
    kind, k, L = case["kind"], case["k"], case["L"]
    if kind in ("front", "image"):
        a, m, t = ctx.cosupport_median(s["rgb"], case["p"], case["p"] / 4.0, s["om"], TAU_FRAC,
                                       precision=case["precision"], alpha=s["alpha"], out=s["masks"], tau=s["tau"])
        if kind == "front":
            return a, m, t
        ll = ctx.label_loglik(s["rgb"], m, k, s["pix"], s["lab"], L, _params(case), out=s["out"])
        return a, m, t, ll
    if kind == "loglik":
        if case["form"] == "soft":
            return ctx.label_loglik_soft(s["rgb"], s["alpha"], SIGMA_IOTA, s["pix"], s["lab"], L, _params(case),
                                         out=s["out"])
        return ctx.label_loglik(s["rgb"], s["masks"], k, s["pix"], s["lab"], L, _params(case),
                                pix_subset=s.get("subset"), out=s["out"], joint=case["form"] == "joint")
    if kind == "segment":
        labels, u, st = ctx.segment(s["rgb"], s["ll"], SegmentParams(
            lam=1.0, nu=case["nu"], iterations=case["iters"], precision=case["precision"]), want_u=True)
        return labels, u, st
    if kind == "unsup":
        c = _classes(case)
        ll, cl = ctx.unsupervised_loglik(s["rgb"], s["masks"], k, s["init"][0], s["init"][1],
                                         UnsupParams(colour_classes=c, texture_classes=c, iterations=10))
        labels, u, st = ctx.segment(s["rgb"], ll, SegmentParams(lam=6.0, nu=case["nu"], iterations=case["iters"]),
                                    want_u=True)
        return ll, cl, labels, u, st
    if kind == "fit":
        net = Mlp(ctx, 5 + k, L, s["net"])
        net.fit_output_bias(s["ell"])
        trace = net.train(s["x"], s["ell"], s["order"], case["batch"], 3e-3)
        return net.params(), trace
    if kind == "infer":
        return s["mlp"].infer(s["rgb"], s["alpha"], out=s["out"])
    out, n = s["mlp"].infer_fallback(s["rgb"], s["alpha"], s["masks"], k, s["pix"], s["lab"], _params(case),
                                     margin=2.0, out=s["out"])
    return out, n


def work(case):
    """Bytes of the inputs and outputs, each once, and the operations of the
    definition (a pair: location 5, colour 8, three per 32-bit mask word,
    exponent, scale and sum 6)."""
    N, p, k, L, M = case["H"] * case["W"], case["p"], case["k"], case["L"], case["M"]
    words = (k + 63) // 64
    kind = case["kind"]
    front_b, front_f = 12 * N + 4 * k * p * p + 4 * N * k + 8 * N * words, 2.0 * N * k * p * p
    rows = case["subset"] or N
    texture = 3 * ((k + 31) // 32) if case["form"] == "sum" else 0
    soft = case["form"] == "soft" and kind == "loglik"
    ll_b = 12 * rows + (4 * k if soft else 8 * words) * rows + 8 * M + 4 * rows * L
    ll_f = float(rows) * M * (19 + texture) + (0.0 if texture else 4.0 * rows * L * k)
    if kind == "front":
        return {"bytes": front_b, "flops": front_f}
    if kind == "image":
        return {"bytes": front_b + 8 * M + 4 * N * L, "flops": front_f + ll_f}
    if kind == "loglik":
        return {"bytes": ll_b, "flops": ll_f}
    seg_b, seg_f = 12 * N + 8 * N * L + 4 * N, 40.0 * N * L * case["iters"]
    if kind == "segment":
        return {"bytes": seg_b, "flops": seg_f}
    if kind == "unsup":
        c = _classes(case)
        return {"bytes": 12 * N + 8 * N * words + seg_b,
                "flops": seg_f + 11.0 * N * c * (8 + 3 * ((k + 31) // 32))}
    net = HID * (5 + k) + HID * HID + HID * L
    if kind == "fit":
        n = case["batch"] * case["steps"]
        return {"bytes": 4 * n * (5 + k + L), "flops": 6.0 * net * n}
    return {"bytes": 12 * N + 4 * N * k + 4 * N * L, "flops": 2.0 * net * N}


# ---- the definitions in 64 bits -----------------------------------------------
def _loglik64(case, s, rows=None):
    """Per-label log-likelihoods of the listed pixels (or all) from the definition."""
    H, W, L, k = case["H"], case["W"], case["L"], case["k"]
    form = case["form"]
    f8 = torch.float64
    if rows is None:
        rows = torch.arange(H * W, device="cuda")
    n = rows.numel()
    flat = s["rgb"].reshape(3, -1).double()
    pix, lab = s["pix"].long(), s["lab"].long()
    out = torch.empty(n, L, device="cuda", dtype=f8)
    tex = torch.empty(n, L, device="cuda", dtype=f8) if form != "sum" else None
    sc2 = 2.0 * 0.05 ** 2
    if form == "soft":
        iota = lambda q: torch.exp(-s["alpha"][q].double() ** 2 / SIGMA_IOTA)  # noqa: E731
    for l in range(L):
        sp = pix[lab == l]
        m = sp.numel()
        ys = torch.stack([(sp % W).to(f8), (sp // W).to(f8)], 1)
        cs = flat[:, sp].t()
        sb = _bits(s["masks"][sp], k) if form != "soft" else None
        if form == "joint":
            rep = (2 * sb.sum(0) >= m).float()
        elif form == "soft":
            rep = iota(sp).sort(0).values[m // 2]
        step = max(1, 48_000_000 // m)
        for a in range(0, n, step):
            q = rows[a:a + step]
            xs = torch.stack([(q % W).to(f8), (q // W).to(f8)], 1)
            x2, y2 = (xs * xs).sum(1, keepdim=True), (ys * ys).sum(1, keepdim=True)
            d2 = torch.addmm(y2.t().expand(q.numel(), m), xs, ys.t(), alpha=-2.0).add_(x2)
            near = d2.min(1, keepdim=True).values
            rho2 = 1.3 ** 2 * near.clamp_min(1.0)
            e = d2.div_(-2.0 * rho2)
            cx = flat[:, q].t()
            c2 = torch.addmm((cs * cs).sum(1)[None, :].expand(q.numel(), m), cx, cs.t(), alpha=-2.0)
            e.sub_(c2.add_((cx * cx).sum(1, keepdim=True)).div_(sc2))
            del c2
            beta = rho2.sqrt()
            if form == "sum":
                xb = _bits(s["masks"][q], k)
                t = torch.addmm(sb.sum(1)[None, :].expand(q.numel(), m), xb, sb.t(), alpha=-2.0)
                e.sub_(t.add_(xb.sum(1, keepdim=True)).double().div_(beta))
                del t
            elif form == "joint":
                tex[a:a + step, l] = -((_bits(s["masks"][q], k) - rep).abs().sum(1).double() / beta[:, 0])
            else:
                tex[a:a + step, l] = -((iota(q) - rep).abs().sum(1) / beta[:, 0])
            out[a:a + step, l] = (torch.logsumexp(e, 1) - math.log(m) - torch.log(2.0 * math.pi * rho2[:, 0])
                                  - 1.5 * math.log(math.pi * sc2))
    if tex is not None:
        out += tex - torch.logsumexp(tex, 1, keepdim=True)
    if case["normalise"]:
        out -= torch.logsumexp(out, 1, keepdim=True)
    return out


def _segment64(case, rgb, ll, lam, nu, iters):
    """(u, energies) of the primal-dual scheme in 64 bits."""
    H, W = case["H"], case["W"]
    L, N = ll.shape[1], H * W
    f = -ll.double().t().reshape(L, H, W)
    r = rgb.double()

    def grad(v):
        gx, gy = torch.zeros_like(v), torch.zeros_like(v)
        gx[..., :, :-1] = v[..., :, 1:] - v[..., :, :-1]
        gy[..., :-1, :] = v[..., 1:, :] - v[..., :-1, :]
        return gx, gy

    def div(px, py):
        d = torch.zeros_like(px)
        d[..., :, :-1] += px[..., :, :-1]
        d[..., :, 1:] -= px[..., :, :-1]
        d[..., :-1, :] += py[..., :-1, :]
        d[..., 1:, :] -= py[..., :-1, :]
        return d

    gx, gy = grad(r)
    mag = (gx * gx + gy * gy).sum(0).sqrt()
    gamma = float(mag.mean())
    rad = 0.5 * lam * torch.exp(-mag / gamma) / (2.0 * gamma)
    u = torch.full((L, H, W), 1.0 / L, device="cuda", dtype=torch.float64)
    ub, px, py, mu = u.clone(), torch.zeros_like(u), torch.zeros_like(u), torch.zeros_like(u)
    m = mb = torch.ones(L, device="cuda", dtype=torch.float64)
    tau_u = 0.2 if nu > 0 else 0.25
    ranks = torch.arange(1, L + 1, device="cuda", dtype=torch.float64)[:, None, None]
    for _ in range(iters):
        gx, gy = grad(ub)
        px, py = px + 0.5 * gx, py + 0.5 * gy
        s = torch.clamp_max(rad / torch.sqrt(px * px + py * py).clamp_min(1e-300), 1.0)
        px, py = px * s, py * s
        step = f - div(px, py)
        if nu > 0:
            mu = (mu + 0.5 * (mb[:, None, None] - ub)).clamp_max(0.0)
            step = step - mu
            mn = (m - (nu + mu.sum((1, 2))) / N).clamp(0.0, 1.0)
            m, mb = mn, 2.0 * mn - m
        v = u - tau_u * step
        z = v.sort(0, descending=True).values
        c = (z.cumsum(0) - 1.0) / ranks
        kk = (z > c).sum(0, keepdim=True)
        un = (v - c.gather(0, kk - 1)).clamp_min(0.0)
        ub, u = 2.0 * un - u, un
    gx, gy = grad(u)
    primal = (u * f).sum() + (rad * (gx * gx + gy * gy).sqrt()).sum() + nu * u.amax((1, 2)).sum()
    lab = u.argmax(0)
    ind = torch.nn.functional.one_hot(lab, L).permute(2, 0, 1).double()
    gx, gy = grad(ind)
    binary = (ind * f).sum() + (rad * (gx * gx + gy * gy).sqrt()).sum() + nu * lab.unique().numel()
    dual = (f - div(px, py) - mu).amin(0).sum()
    if nu > 0:
        dual = dual + (nu + mu.sum((1, 2))).clamp_max(0.0).sum()
    stats = {"primal": float(primal), "binary": float(binary), "dual": float(dual), "gamma": gamma,
             "labels_used": None}
    return u.reshape(L, N).t().contiguous(), stats


def _cluster64(case, s):
    """The unsupervised class log-likelihoods and the colour centroids."""
    k, c = case["k"], _classes(case)
    colours = s["rgb"].reshape(3, -1).t().double()
    bits = _bits(s["masks"], k)
    cc, tc = colours[torch.tensor(s["init"][0], device="cuda").long()], bits[torch.tensor(s["init"][1],
                                                                                       device="cuda").long()]

    def dist(cc, tc):
        dc = torch.stack([((colours - cc[i]) ** 2).sum(1) for i in range(c)], 1)
        dt = torch.stack([(bits - tc[i]).abs().sum(1) for i in range(c)], 1).double()
        return dc, dt

    for _ in range(10):
        dc, dt = dist(cc, tc)
        a, b = dc.argmin(1), dt.argmin(1)
        cc = torch.stack([colours[a == i].mean(0) if bool((a == i).any()) else cc[i] for i in range(c)])
        tc = torch.stack([(2 * bits[b == i].sum(0) >= (b == i).sum()).float() if bool((b == i).any()) else tc[i]
                          for i in range(c)])
    dc, dt = dist(cc, tc)
    dc, dt = -dc / (2.0 * 0.05 ** 2), -dt / 2.0
    ec, et = dc.repeat_interleave(c, 1), dt.repeat(1, c)
    return ec - torch.logsumexp(ec, 1, keepdim=True) + et - torch.logsumexp(et, 1, keepdim=True), cc


def exact(case, seed):
    kind, k, L = case["kind"], case["k"], case["L"]
    s = _inputs(case, seed)
    if kind in ("front", "image"):
        a = _analysed(case, s["rgb"], s["om"], torch.float64)
        b = a.abs().flatten()
        tau = TAU_FRAC * b.kthvalue((b.numel() - 1) // 2 + 1).values
        if kind == "front":
            return a, None, tau.reshape(1)
        s["masks"] = torch.zeros(a.shape[0], (k + 63) // 64, device="cuda", dtype=torch.int64)
        for j in range(k):
            s["masks"][:, j // 64] |= (a[:, j].abs() <= tau).long() << (j % 64)
        return a, None, tau.reshape(1), _loglik64(case, s)
    if kind == "loglik":
        return _loglik64(case, s, s["subset"].long() if case["subset"] else None)
    if kind == "segment":
        u, st = _segment64(case, s["rgb"], s["ll"], 1.0, case["nu"], case["iters"])
        return None, u, st
    if kind == "unsup":
        ll, cc = _cluster64(case, s)
        u, st = _segment64(case, s["rgb"], ll, 6.0, case["nu"], case["iters"])
        return ll, {"colour_centroids": cc, "texture_centroids": None, "colour_labels": None,
                    "texture_labels": None}, None, u, st
    if kind == "fit":
        x, ell = s["x"].double(), s["ell"].double()
        t = torch.maximum(ell, ell.max(1, keepdim=True).values - CLIP)
        flat = s["net"].double()
        flat[-L:] = t.mean(0)
        flat.requires_grad_(True)
        opt = torch.optim.Adam([flat], lr=3e-3)
        trace = []
        for idx in s["order"].long().reshape(case["steps"], case["batch"]):
            ps = _net_split(flat, k, L)
            loss = ((_net_hidden(ps, x[idx]) @ ps[4].t() + ps[5] - t[idx]) ** 2).mean()
            opt.zero_grad()
            loss.backward()
            opt.step()
            trace.append(loss.detach())
        return flat.detach(), torch.stack(trace)
    if kind == "infer":
        ps = _net_split(s["net"].double(), k, L)
        N = case["H"] * case["W"]
        y = [_net_hidden(ps, _rows(case, s["rgb"], s["alpha"], q).double()) @ ps[4].t() + ps[5]
             for q in torch.arange(N, device="cuda").split(1 << 19)]
        return torch.cat(y)
    return None  # which pixels are unsure is decided on BF16 outputs: no 64-bit value
