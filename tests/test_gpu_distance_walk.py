"""The distance transform's row walk over far and few samples: rows of one block
to many runs of blocks, ragged last blocks and columns of many segments, in the
full and the listed pass; and sample counts around one and two levels of done
counters.  Bars as in test_gpu_parity; listed rows equal the full ones."""
import numpy as np
import pytest
from test_gpu_parity import _ll_check, _loglik_both, ctx  # noqa: F401

import oracle
from workloads import make_workload

pytestmark = pytest.mark.gpu


def _case(H, W, M, seed):
    w = make_workload("walk", H=H, W=W, R=2, p=3, k=20, seed=seed, per_region=1)
    rng = np.random.default_rng(seed)
    # label 0 at the left end, label 1 at the right, label 2 anywhere
    pix = [np.array([0, w.N - W]), np.array([W - 1, w.N - 1]), rng.integers(0, w.N, M - 4)]
    w.sample_pix = np.concatenate(pix).astype(np.int32)
    w.sample_label = np.repeat([0, 1, 2], [2, 2, M - 4]).astype(np.int32)
    w.L = 3
    return w


@pytest.mark.parametrize("H,W", [(40, 16), (33, 17), (9, 144), (7, 161), (5, 300), (4, 1501), (512, 20), (513, 20), (700, 24)])
def test_far_samples(ctx, H, W):  # noqa: F811
    w = _case(H, W, 7, seed=H + W)
    masks, _, _ = oracle.full_masks(w)
    full, ref = _loglik_both(ctx, w, masks)
    _ll_check(full, ref)
    pix = np.random.default_rng(W).integers(0, w.N, w.N // 9).astype(np.int32)
    got, ref = _loglik_both(ctx, w, masks, pix=pix)
    _ll_check(got, ref)


@pytest.mark.parametrize("M", [255, 256, 257, 4096, 4097, 8449])
def test_sample_counts(ctx, M):  # noqa: F811
    w = _case(24, 40, M, seed=M)
    masks, _, _ = oracle.full_masks(w)
    for _ in range(2):
        got, ref = _loglik_both(ctx, w, masks)
        _ll_check(got, ref)
