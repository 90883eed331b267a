"""The one-launch solve where its tiles cannot wait for each other: a refused
arrival takes the tile form (the same arithmetic), a word that is not waited for
ends without a result and says so; solves on two streams at a time and beside
other work.  Every launch ends by itself.  Bars as in test_gpu_segment."""
import ctypes
import threading

import numpy as np
import pytest
import torch
from test_gpu_segment import _check, _synthetic_term, dev

from workloads import make_workload

pytestmark = pytest.mark.gpu


def _ctx(arrive=0.02, words=1, error=0):
    from paper_1312_4746_amd import Context, lib
    c = Context(0)
    f = lib().cs_segment_waits
    f.argtypes = [ctypes.c_void_p, ctypes.c_double, ctypes.c_int, ctypes.c_int]
    assert f(c._h, arrive, words, error) == 0
    return c


def _case(H, W, L, seed):
    w = make_workload("seg_waits", H=H, W=W, R=max(2, min(L, 6)), p=3, k=8, seed=seed, per_region=1)
    w.L = L
    w.region = w.region % L
    return w, _synthetic_term(w, seed=L)


def _params(nu, iters):
    from paper_1312_4746_amd import SegmentParams
    return SegmentParams(lam=1.5, nu=nu, iterations=iters, precision="fp32")


def _solve(c, w, ll, prm, stats=True):
    lab, u, st = c.segment(dev(w.rgb), dev(ll), prm, want_u=True, stats=stats)
    return lab.cpu(), u.cpu(), st


@pytest.mark.parametrize("H,W,L,nu", [(121, 150, 6, 0.0), (40, 61, 16, 0.0), (90, 151, 3, 20.0), (20, 20, 2, 0.0)])
def test_refused_arrival_takes_the_tile_form(H, W, L, nu):
    w, ll = _case(H, W, L, 23)
    c = _ctx(arrive=-1.0)
    _check(c, w.rgb, ll, 1.5, nu, 9, "fp32")
    prm = _params(nu, 9)
    got = _solve(c, w, ll, prm)
    c.profile_only("pd_iter")
    c.profile_enable(True)
    _solve(c, w, ll, prm)
    assert c.profile_read("pd_iter")[1] > 1
    c.profile_enable(False)
    c2 = _ctx()
    ref = _solve(c2, w, ll, prm)
    if nu == 0.0:
        assert torch.equal(got[1], ref[1]) and torch.equal(got[0], ref[0]) and got[2] == ref[2]
    c2.close()
    c.close()


@pytest.mark.parametrize("H,W,L,nu", [(121, 150, 6, 0.0), (90, 151, 3, 20.0)])
def test_lost_words_are_reported(H, W, L, nu):
    from paper_1312_4746_amd import CosparseError
    w, ll = _case(H, W, L, 24)
    c = _ctx(words=0)
    with pytest.raises(CosparseError) as e:
        _solve(c, w, ll, _params(nu, 9))
    assert e.value.code == 3
    lab, u, _ = _solve(c, w, ll, _params(nu, 9), stats=False)
    assert bool((lab == -1).all()) and bool(u.isnan().all())
    from paper_1312_4746_amd import lib
    assert lib().cs_segment_waits(c._h, 0.02, 1, 0) == 0
    _check(c, w.rgb, ll, 1.5, nu, 9, "fp32")
    c.close()


@pytest.mark.parametrize("error,falls_back", [(720, True), (801, True), (1, False), (2, False), (719, False)])
def test_errors_of_the_launch(error, falls_back):
    """A launch too large for the device (720) or not supported (801) takes the
    tile form; any other error is the call's."""
    from paper_1312_4746_amd import CosparseError
    w, ll = _case(40, 61, 3, 29)
    c = _ctx(error=error)
    if falls_back:
        _check(c, w.rgb, ll, 1.5, 0.0, 9, "fp32")
    else:
        with pytest.raises(CosparseError) as e:
            _solve(c, w, ll, _params(0.0, 9))
        assert e.value.code == 3
    c.close()


def test_without_stats():
    w, ll = _case(121, 150, 6, 25)
    c = _ctx()
    a, b = _solve(c, w, ll, _params(0.0, 30)), _solve(c, w, ll, _params(0.0, 30), stats=False)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    c.close()


def test_two_contexts_two_streams():
    cases = [_case(160, 241, 10, 26), _case(131, 200, 16, 27)]
    prms = [_params(0.0, 60), _params(15.0, 60)]
    ctxs = [_ctx(), _ctx()]
    alone = [_solve(ctxs[i], *cases[i], prms[i]) for i in range(2)]
    out, errors = [None, None], []

    def run(i):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                out[i] = [_solve(ctxs[i], *cases[i], prms[i]) for _ in range(8)]
        except Exception as e:  # noqa: BLE001
            errors.append(e)

    threads = [threading.Thread(target=run, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for r in out[0]:
        assert torch.equal(r[0], alone[0][0]) and torch.equal(r[1], alone[0][1])
    for r in out[1]:  # (a label cost: the forms add the tiles' sums in another order)
        assert float((r[1] - alone[1][1]).abs().max()) <= 1e-3
    for c in ctxs:
        c.close()


def test_beside_other_work():
    w, ll = _case(321, 481, 10, 28)
    c = _ctx()
    alone = _solve(c, w, ll, _params(0.0, 60))
    a = torch.randn(4096, 4096, device="cuda")
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        for _ in range(12):
            a @ a
    r = _solve(c, w, ll, _params(0.0, 60))
    torch.cuda.synchronize()
    assert torch.equal(r[0], alone[0]) and torch.equal(r[1], alone[1])
    c.close()


@pytest.mark.parametrize("nu,top", [(1e5, 3), (3e5, 3), (3e5, 6)])
def test_label_cost_sums_keep_every_bit(nu, top):
    """450 x 480 with 3 labels has the same tiles in both forms, whose FP64 sums of
    the multipliers differ by the order of additions alone: 2^-53 for each of the
    240 tiles and 400 iterations of a sum that the dual energy contains.  The data
    term's strength varies by rows, so that a tile's sum spans more binades than
    37 bits hold."""
    w, ll = _case(450, 480, 3, 30)
    rows = np.exp(np.random.default_rng(1).uniform(-9, top, w.H)).astype(np.float32)
    ll = ll * np.repeat(rows, w.W)[:, None]
    prm = _params(nu, 400)
    c, c2 = _ctx(), _ctx(arrive=-1.0)
    c.profile_only("pd_iter")
    c.profile_enable(True)
    got = _solve(c, w, ll, prm)
    assert c.profile_read("pd_iter")[1] == 1
    c.profile_enable(False)
    ref = _solve(c2, w, ll, prm)
    print(got[2], ref[2])
    assert abs(got[2]["dual"] - ref[2]["dual"]) <= 240 * 400 * 2.0 ** -53 * abs(ref[2]["dual"])
    assert float((got[1] - ref[1]).abs().max()) <= 2.0 ** -24
    c.close()
    c2.close()
