"""Centroid of the registration points, at fewer and more blocks than the
1024 lanes that sum it: seen through the pose of a multi-start turn about it."""
import math

import numpy as np
import pytest

import scenegen as sg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cv():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2410_21149_amd as m
    return m


@pytest.mark.parametrize("vs", [0.1, 0.05, 0.025])
def test_centroid_of_the_points(cv, vs):
    import torch
    w = sg.tiny()
    dev = torch.from_numpy(w.frames(0, 6)).cuda()
    ctx = cv.Context(voxel_size=vs, trunc_vox=4, max_range=5.0, d_max=2.0 if vs >= 0.05 else 1.0,
                     block_capacity=16384, max_iter=0, w_reg=1.0)
    s = ctx.submap_create()
    ctx.integrate_depth_batch(s, dev, w.cam.K, w.poses[:6])
    ctx.update_esdf(s)
    n_blocks = ctx.submap_info(s)["n_blocks"]
    assert (n_blocks > 1024) == (vs == 0.025), n_blocks
    p = ctx.export_points(s).astype(np.float64).mean(axis=0)
    half = np.diag([-1.0, -1.0, 1.0, 1.0])

    def turned(c):  # half a turn about the vertical through c
        T = half.copy()
        T[:2, 3] = 2 * c[:2]
        return T

    # from the half turn about the centroid, the second start turns back: the
    # identity, whose cost on the submap itself is the least
    T, cost, st = ctx.align_multistart(s, s, turned(p), n_starts=2)
    assert st["best_start"] == 1
    # n points of up to 10 m summed in binary64: within n 2^-52 10 m, twice
    assert np.max(np.abs(T - np.eye(4))) <= 2 * st["n_points"] * 2.0 ** -52 * 10 + 1e-14 * math.pi
    ctx.close()


@pytest.mark.parametrize("precision", ["FP32", "FP16"])
def test_points_into_room_of_any_size(cv, precision):
    """Points extracted into no room, into enough left by an earlier extraction, and
    into too little: the same as from a submap that extracts for the first time, and
    the oracle's (positions within one rounding of the edge's division, 2^-22 of a
    voxel, and of the sum, 2^-24 of 8 m)."""
    import oracle as orc
    import torch
    w = sg.tiny()
    fr = w.frames(0, 12)
    dev = torch.from_numpy(fr).cuda()
    kw = dict(voxel_size=0.05, trunc_vox=4, max_range=5.0, d_max=2.0, block_capacity=16384, w_reg=1.0,
              precision=getattr(cv, precision))
    ctx = cv.Context(**kw)
    s = ctx.submap_create()
    for n in (1, 2, 12, 3, 3):  # none, perhaps short, short, plenty twice
        print("points of", n, "frames", flush=True)
        ctx.submap_reset(s)
        ctx.integrate_depth_batch(s, dev[:n], w.cam.K, w.poses[:n])
        got = ctx.export_points(s)
        t = ctx.submap_create()
        ctx.integrate_depth_batch(t, dev[:n], w.cam.K, w.poses[:n])
        first = ctx.export_points(t)
        assert len(got) > 0 and np.array_equal(got, first)
        ref = orc.Submap(orc.Params(vs=0.05, w_reg=1.0, fp16=precision == "FP16"))
        for f in range(n):
            ref.integrate(fr[f], w.cam.K, w.poses[f])
        exp = np.asarray(ref.iso_points(), np.float64).reshape(-1, 3)
        assert len(exp) == len(got)
        assert np.abs(got.astype(np.float64) - exp).max() <= 0.05 * 2.0 ** -22 + 8 * 2.0 ** -24
    ctx.close()
