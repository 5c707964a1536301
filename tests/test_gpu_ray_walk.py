"""The raycast integrator's one-walk frames (accumulators by box block) against its
two-walk frames, which a pool of fewer blocks than the box takes: the same blocks in
the same order, the same contribution counts, W equal (integer counts with constant
weights) and D within the rounding of sums taken in another order, over both weights,
carving on and off, ragged image sizes, voxels from small to coarse; and a frame that
overflows leaves the accumulators clean."""
import numpy as np
import pytest

import scenegen as sg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cv():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_21149_amd as cv
    return cv


def _ctx(cv, vs, **kw):
    base = dict(voxel_size=vs, trunc_vox=4, max_range=5.0, d_max=10 * vs, integrator=cv.RAYCAST)
    base.update(kw)
    return cv.Context(**base)


@pytest.mark.parametrize("weight", ["WEIGHT_CONSTANT", "WEIGHT_INV_DEPTH2"])
@pytest.mark.parametrize("vs,rows,cols,carve", [
    (0.05, 480, 640, 1), (0.05, 480, 640, 0), (0.05, 33, 47, 1), (0.05, 1, 1, 1), (0.20, 17, 640, 1), (0.03, 100, 15, 0),
])
def test_one_walk_equals_two(cv, vs, rows, cols, carve, weight):
    import torch
    w = sg.room(n_frames=3)
    fr = np.ascontiguousarray(w.frames()[:, :rows, :cols])
    fr[1, ::3] = 0.0
    dev = torch.from_numpy(fr).cuda()
    out = []
    cap = 1 << 16
    for _ in range(2):
        print("rays", vs, rows, cols, carve, weight, "pool", cap, flush=True)
        ctx = _ctx(cv, vs, block_capacity=cap, ray_carve=carve, weight_mode=getattr(cv, weight))
        s = ctx.submap_create()
        for _ in range(2):  # existing blocks the second time
            for f in range(3):
                ctx.integrate_depth(s, dev[f], w.cam.K, w.poses[f])
        out.append((ctx.export_blocks(s), ctx.submap_info(s)["n_updates"]))
        ctx.close()
        cap = max(1, len(out[0][0]["keys"]))  # the blocks needed and no more: fewer than the box has
    (a, na), (b, nb) = out
    assert na == nb and np.array_equal(a["keys"], b["keys"])
    Wa, Wb = a["W"].astype(np.float64), b["W"].astype(np.float64)
    # binary64 sums of a frame in another order, each rounded once to binary32, six frames
    if weight == "WEIGHT_CONSTANT":
        assert np.array_equal(Wa, Wb)
    else:
        assert np.abs(Wa - Wb).max() <= 6 * 2.0 ** -23 * Wa.max()
    assert np.abs(a["D"].astype(np.float64) - b["D"]).max() <= 6 * 2.0 ** -22 * 4 * vs


def test_overflowing_frame_leaves_no_sums(cv):
    """The pool holds the box of one frame, so frames take one walk until a far one
    overflows it; the frames after that are as if it had not come."""
    import torch
    w = sg.tiny(n_frames=2)
    fr = torch.from_numpy(w.frames()).cuda()
    far = []
    for k in range(64):  # the same view from positions that share no block
        T = np.array(w.poses[0], np.float64)
        T[:3, 3] += [40.0 * k, 0.0, 0.0]
        far.append(T)
    probe = _ctx(cv, 0.05, block_capacity=1 << 16)
    s = probe.submap_create()
    probe.integrate_depth(s, fr[0], w.cam.K, far[0])
    one = probe.submap_info(s)["n_blocks"]
    probe.close()
    cap = 6000
    ctx = _ctx(cv, 0.05, block_capacity=cap)
    ref = _ctx(cv, 0.05, block_capacity=1 << 16)
    a, b = ctx.submap_create(), ref.submap_create()
    n = 0
    print("overflow after about", cap // one, "frames", flush=True)
    for T in far:
        try:
            ctx.integrate_depth(a, fr[0], w.cam.K, T)
        except cv.CovoxError as e:
            assert e.code == cv.EPOOL_FULL
            break
        ref.integrate_depth(b, fr[0], w.cam.K, T)
        n += 1
    assert 0 < n < len(far)
    for T in far[:2]:
        ctx.integrate_depth(a, fr[0], w.cam.K, T)
        ref.integrate_depth(b, fr[0], w.cam.K, T)
    ea, eb = ctx.export_blocks(a), ref.export_blocks(b)
    assert np.array_equal(ea["keys"], eb["keys"])
    assert np.array_equal(ea["W"], eb["W"])
    assert np.abs(ea["D"].astype(np.float64) - eb["D"]).max() <= 6 * 2.0 ** -22 * 0.2
    ctx.close()
    ref.close()
