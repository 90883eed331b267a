"""The clustering launches at the class counts, mask widths and image sizes
where their variants change: 4 or 16 classes, 1 to 4 mask words, one or several
pixels per thread (512 workgroups of 256).  Bars as in test_gpu_unsup."""
import numpy as np
import pytest
from test_gpu_unsup import _case, ctx  # noqa: F401

from workloads import make_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,k,Kc,Kt", [(41, 67, 64, 8, 8), (41, 67, 65, 5, 12), (37, 53, 200, 4, 5),
                                         (33, 47, 256, 16, 4), (1, 9, 1, 2, 2), (300, 467, 130, 4, 3),
                                         (363, 362, 40, 6, 5)])
def test_variants(ctx, H, W, k, Kc, Kt):  # noqa: F811
    w = make_workload("us_parts", H=H, W=W, R=2, p=3, k=8, seed=33, per_region=1)
    w.k = k
    rng = np.random.default_rng(k)
    proto = rng.random((6, k)) < 0.4
    bits = proto[rng.integers(0, 6, w.N)] ^ (rng.random((w.N, k)) < 0.2)
    words = np.zeros((w.N, (k + 63) // 64), np.uint64)
    for j in range(k):
        words[:, j // 64] |= bits[:, j].astype(np.uint64) << np.uint64(j % 64)
    _case(ctx, w, words, Kc, Kt, 4, seed=3)
