"""The field of an alignment read from tiles or through its page: the same bits, over
every solver, launch shape and call, with points inside the field, over its edges and
outside it; and whatever the library chooses for few points and many."""
import numpy as np
import pytest

import oracle as orc
import scenegen as sg

pytestmark = pytest.mark.gpu


def _moved(x, y):
    T = orc.se3_exp(np.array([0.02, -0.01, 0.01, 0.01, -0.01, 0.02]))
    T[:2, 3] += [x, y]
    return T


STARTS = [_moved(0, 0), _moved(2.0, -1.5), _moved(3.9, 0.3), _moved(300.0, 0)]


@pytest.mark.parametrize("rows", [4, 120])  # one segment of points, and several
@pytest.mark.parametrize("lm,dof,lanes,pairs", [(False, 6, 256, 1), (True, 6, 512, 1), (False, 4, 256, 2), (True, 4, 512, 2)])
def test_tiles_and_pages_give_the_same_bits(monkeypatch, rows, lm, dof, lanes, pairs):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_21149_amd as cv
    w = sg.tiny()
    dev = torch.from_numpy(w.frames(0, 12)).cuda()
    part = dev.clone()
    part[:, rows:] = 0.0
    got = {}
    for field in ("tiles", "pages", "by rule"):
        monkeypatch.setenv("COVOX_ALIGN_FIELD", field)
        ctx = cv.Context(block_capacity=4096, w_reg=1.0, n_min=20, voxel_size=0.05, trunc_vox=4, max_range=5.0, d_max=2.0,
                         align_dof=dof, align_solver=cv.LEVENBERG_MARQUARDT if lm else cv.GAUSS_NEWTON)
        ctx.set_tuning(align_threads=lanes, align_points_per_step=pairs)
        A, B = ctx.submap_create(), ctx.submap_create()
        for f in range(12):
            ctx.integrate_depth(A if f % 2 == 0 else B, (dev if f % 2 == 0 else part)[f], w.cam.K, w.poses[f])
        ctx.update_esdf_batch([A, B])
        print(field, "points", len(ctx.export_points(B)), flush=True)
        out = []
        for T0 in STARTS:
            T, c, st = ctx.align_submaps(A, B, T0)
            out += [T, c, st["n_used"], st["solves"], st["status"], ctx.normal_equations(A, B, T0)]
        T, c, st = ctx.align_batch([(A, B, T0) for T0 in STARTS] + [(B, A, STARTS[0])], 3)
        out += [T, c, [s["n_used"] for s in st]]
        S = ctx.align_prepare([(A, B, T0) for T0 in STARTS], 2)
        S.launch()
        T, c, st = S.collect()
        S.close()
        out += [T, c, [s["n_used"] for s in st]]
        x, st = ctx.pgo_solve([A, B], np.array([[0.0, 0, 0, 0], [0.02, -0.01, 0.01, 0.01]]), [(0, 1), (1, 0)], [])
        out += [x, st["cost_init"], st["cost_final"]]
        got[field] = out
        ctx.close()
    used = got["tiles"][2]
    assert used > 100 and 0 < got["tiles"][14] < used  # all inside, some over the edge
    for field in ("pages", "by rule"):
        for k, (a, b) in enumerate(zip(got["tiles"], got[field])):
            assert np.array_equal(a, b), (field, k)
