"""The benchmark's segmentation leg names the form that ran (from its launches) and
states fractions of peaks that cannot pass them."""
import argparse

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("config,kernel", [(1, "k_pd_resident"), (3, "k_pd_tile")])
def test_form_and_fractions(config, kernel):
    import bench
    args = argparse.Namespace(no_cpu=True, seg_iters=24, seg_lambda=1.0)
    line = bench.segment_line(args, config)
    r = line["roofline"]
    assert r["kernel"] == kernel and (r["launches"] == 1) == (kernel == "k_pd_resident")
    assert 0 < r["frac"] < 1 and r["frac"] == max(r["alu_frac"], r["hbm_frac"])
