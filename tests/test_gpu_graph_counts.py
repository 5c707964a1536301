"""Block counts after graph replays: the host's bound on them, and what is decided from
it, hold for the replay that is still running, not only for the one before."""
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


KW = dict(voxel_size=0.05, trunc_vox=4, max_range=5.0, d_max=2.0)


def _busy():
    """Some milliseconds of work on the stream, so that what is enqueued behind it waits."""
    import torch
    a = torch.full((4096, 4096), 1e-3, device="cuda")
    for _ in range(40):
        a = a @ a
    return a


def _far_poses(w, n):
    """Camera poses 30 m apart: every frame adds its own blocks."""
    out = np.repeat(np.array(w.poses[:1], np.float64), n, axis=0)
    out[:, 0, 3] += 30.0 * np.arange(n)
    return out


@pytest.mark.parametrize("precision", ["FP32", "FP16"])
def test_frame_behind_a_replay_that_fills_the_pool(cv, precision):
    """A replay over empty images, then one over full ones that leaves less room than
    the next frame needs, and that frame at once: refused, and nothing of it entered."""
    import torch
    w = sg.tiny()
    n = 24
    full = torch.from_numpy(np.repeat(w.frames(0, 1), n + 1, axis=0)).cuda()
    poses = _far_poses(w, n + 1)
    kw = dict(precision=getattr(cv, precision), **KW)
    ctx = cv.Context(block_capacity=1 << 17, **kw)
    r = ctx.submap_create()
    ctx.integrate_depth_batch(r, full[:n], w.cam.K, poses[:n])
    held = ctx.submap_info(r)["n_blocks"]
    want = ctx.export_blocks(r)["keys"]
    ctx.integrate_depth(r, full[n], w.cam.K, poses[n])
    total = ctx.submap_info(r)["n_blocks"]
    ctx.close()
    assert held > 5000 and total > held + 100

    cap = (held + total) // 2
    ctx = cv.Context(block_capacity=cap, **kw)
    s = ctx.submap_create()
    buf = torch.zeros_like(full[:n])
    ctx.graph_begin()
    ctx.submap_reset(s)
    for f in range(n):
        ctx.integrate_depth(s, buf[f], w.cam.K, poses[f])
    g = ctx.graph_end()
    g.launch()
    ctx.sync()
    assert ctx.submap_info(s)["n_blocks"] == 0
    buf.copy_(full[:n])
    ctx.sync()
    busy = _busy()
    g.launch()
    code = cv.OK
    try:
        ctx.integrate_depth(s, full[n], w.cam.K, poses[n])
    except cv.CovoxError as e:
        code = e.code
    info = ctx.submap_info(s)
    print("blocks %d of %d, call %d, status %d" % (held, cap, code, info["status"]), flush=True)
    assert cv.EPOOL_FULL in (code, info["status"])
    assert info["n_blocks"] == held
    assert np.array_equal(ctx.export_blocks(s)["keys"], want)
    del busy
    g.close()
    ctx.close()
