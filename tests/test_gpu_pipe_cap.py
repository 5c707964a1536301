"""Sequences whose ESDF passes may run few workgroups at once, which then take longer
segments: the calls in order, bit for bit, from the longest segments to the shortest, at
the widest halo and a narrow one, riding with single frames and with batches."""
import numpy as np
import pytest

import scenegen as sg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_max,precision", [(2.8, "FP32"), (0.4, "FP16")])
@pytest.mark.parametrize("every", [1, 4])
def test_capped_passes_equal_the_calls_in_order(every, d_max, precision):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_21149_amd as cv
    w = sg.tiny()
    dev = torch.from_numpy(w.frames(0, 12)).cuda()
    kw = dict(voxel_size=0.05, trunc_vox=4, max_range=5.0, d_max=d_max, block_capacity=1 << 17,
              precision=getattr(cv, precision))
    ref = cv.Context(**kw)
    r = ref.submap_create()
    for f in range(0, 12, every):
        ref.integrate_depth_batch(r, dev[f:f + every], w.cam.K, w.poses[f:f + every])
        ref.update_esdf(r)
    want = ref.export_blocks(r)
    ref.close()
    ctx = cv.Context(**kw)
    s = ctx.submap_create()
    for cap in (1, 16, 64, 200, 700):
        print("cap", cap, flush=True)
        ctx.set_tuning(edt_pipe_max_workgroups=cap)
        ctx.submap_reset(s)
        ctx.map_sequence(s, dev, w.cam.K, w.poses[:12], esdf_every=every)
        got = ctx.export_blocks(s)
        for k in ("keys", "D", "W"):
            assert np.array_equal(got[k], want[k]), k
        assert np.array_equal(got["phi"], want["phi"], equal_nan=True)
    ctx.close()
