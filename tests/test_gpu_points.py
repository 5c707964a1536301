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
