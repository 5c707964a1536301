"""Alignments that end before their cap: a problem alone in one workgroup, launch by
launch with the rest not enqueued, and in a graph that holds every launch, all give the
same bits, whether the problem ends at its first evaluation, converges or never does."""
import numpy as np
import pytest

import oracle as orc
import scenegen as sg

pytestmark = pytest.mark.gpu

FAR = np.array([[1, 0, 0, 500.0], [0, 1, 0, 0], [0, 0, 1, 0], [0, 0, 0, 1.0]])  # outside the field: degenerate
NEAR = orc.se3_exp(np.array([0.02, -0.01, 0.01, 0.01, -0.01, 0.02]))


@pytest.fixture(scope="module")
def maps():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2410_21149_amd as cv
    w = sg.tiny()
    dev = torch.from_numpy(w.frames(0, 12)).cuda()
    ctx = cv.Context(block_capacity=4096, w_reg=1.0, voxel_size=0.05, trunc_vox=4, max_range=5.0, d_max=2.0)
    A = ctx.submap_create()
    for f in range(0, 12, 2):
        ctx.integrate_depth(A, dev[f], w.cam.K, w.poses[f])
    ctx.update_esdf(A)
    moving = {}
    for rows in (3, 10, 120):
        B = moving[rows] = ctx.submap_create()
        part = dev.clone()
        part[:, rows:] = 0.0
        for f in range(1, 12, 2):
            ctx.integrate_depth(B, part[f], w.cam.K, w.poses[f])
    yield cv, ctx, A, moving
    ctx.close()


def _stats(r):
    T, c, st = r
    return T, c, [{k: s[k] for k in ("n_points", "n_used", "iterations", "status", "solves")} for s in st]


@pytest.mark.parametrize("lm", [False, True])
@pytest.mark.parametrize("rows,segments", [(3, 1), (10, 2), (120, 16)])  # of 1024 points
def test_same_bits_however_early_it_ends(maps, rows, segments, lm):
    cv, ctx, A, moving = maps
    B = moving[rows]
    ctx.set_params(n_min=20, align_solver=cv.LEVENBERG_MARQUARDT if lm else cv.GAUSS_NEWTON)
    n = len(ctx.export_points(B))
    print("points", n, flush=True)
    assert -(-n // 1024) == segments
    for cap in (0, 1, 30, 64, 200):
        ctx.set_params(max_iter=cap)
        for T0 in (FAR, NEAR):
            one = ctx.align_submaps(A, B, T0)
            one = _stats((one[0][None], np.array([one[1]]), [one[2]]))
            if T0 is FAR:
                assert one[2][0]["status"] == (cv.NOT_CONVERGED if cap == 0 else cv.EDEGENERATE)
            # with a problem that goes on, alone in a set, twice, and replayed
            T, c, st = _stats(ctx.align_batch([(A, B, T0), (A, B, NEAR)], 1))
            assert np.array_equal(T[0], one[0][0]) and c[0] == one[1][0] and st[0] == one[2][0]
            S = ctx.align_prepare([(A, B, T0)], 1)
            ctx.graph_begin()
            S.launch()
            g = ctx.graph_end()
            for launch in (S.launch, g.launch, S.launch, g.launch):
                launch()
                T, c, st = _stats(S.collect())
                assert np.array_equal(T, one[0]) and np.array_equal(c, one[1]) and st == one[2]
            g.close()
            S.close()
    ctx.set_params(max_iter=30, n_min=100, align_solver=cv.GAUSS_NEWTON)
