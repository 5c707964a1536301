"""Column passes of the exact ESDF at the radii and segment lengths where their
search and staging change: R around multiples of four and eight (offsets a
step, halo blocks), segments of one block, a few, and the library's choice."""
import numpy as np
import pytest

import oracle as orc
import scenegen as sg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cv():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2410_21149_amd as m
    return m


@pytest.mark.parametrize("R", [1, 3, 4, 5, 8, 9, 16, 31, 32, 33, 55, 56])
def test_radius_and_segment_edges(cv, R):
    import torch
    w = sg.tiny()
    frames = w.frames(0, 3)
    dev = torch.from_numpy(frames).cuda()
    P = dict(trunc_vox=4, max_range=5.0)
    ref = orc.Submap(orc.Params(vs=0.05, d_max=0.05 * R, **P))
    for f in range(3):
        ref.integrate(frames[f], w.cam.K, w.poses[f])
    ref.update_esdf()
    r = ref.export()["phi"]
    m = ~np.isnan(r)
    ctx = cv.Context(voxel_size=0.05, d_max=0.05 * R, block_capacity=4096, **P)
    s = ctx.submap_create()
    ctx.integrate_depth_batch(s, dev, w.cam.K, w.poses[:3])
    ctx.set_tuning(esdf_full_recompute=1)
    first = None
    for seg in (0, 1, 3, 64):
        ctx.set_tuning(edt_col_seg=seg)
        ctx.update_esdf(s)
        g = ctx.export_blocks(s)["phi"]
        assert np.array_equal(np.isnan(g), ~m), seg
        assert np.max(np.abs(g[m] - r[m])) <= 1e-4, seg
        first = g if first is None else first
        assert np.array_equal(g[m], first[m]), seg
    # many submaps in one launch, and envelopes for either pass
    t = ctx.submap_create()
    ctx.integrate_depth_batch(t, dev, w.cam.K, w.poses[:3])
    big = np.iinfo(np.int64).max
    for y, z in ((big, big), (0, big), (big, 0), (0, 0)):
        ctx.set_tuning(edt_col_seg=0, edt_y_env_min_cols=y, edt_z_env_min_cols=z)
        ctx.update_esdf_batch([s, t])
        for q in (s, t):
            assert np.array_equal(ctx.export_blocks(q)["phi"][m], first[m]), (y, z)
    ctx.close()
