"""Registration points without a weight limit: an edge to a block that is not there is
no edge, whatever the limit (the oracle's points, positions within one rounding of the
edge's division, 2^-22 of a voxel, and of the sum, 2^-24 of 8 m)."""
import numpy as np
import pytest

import oracle as orc
import scenegen as sg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["FP32", "FP16"])
@pytest.mark.parametrize("w_reg", [0.0, -1.0, -1e300, -np.inf])
def test_points_without_a_weight_limit(w_reg, precision):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_21149_amd as cv
    w = sg.tiny()
    fr = w.frames(0, 3)
    ctx = cv.Context(voxel_size=0.05, trunc_vox=4, max_range=5.0, d_max=2.0, block_capacity=16384, w_reg=w_reg,
                     precision=getattr(cv, precision))
    s = ctx.submap_create()
    ctx.integrate_depth_batch(s, torch.from_numpy(fr).cuda(), w.cam.K, w.poses[:3])
    got = ctx.export_points(s).astype(np.float64)
    ctx.close()
    ref = orc.Submap(orc.Params(vs=0.05, w_reg=w_reg, fp16=precision == "FP16"))
    for f in range(3):
        ref.integrate(fr[f], w.cam.K, w.poses[f])
    exp = np.asarray(ref.iso_points(), np.float64).reshape(-1, 3)
    assert len(exp) > 1000 and len(got) == len(exp)
    assert np.abs(got - exp).max() <= 0.05 * 2.0 ** -22 + 8 * 2.0 ** -24
