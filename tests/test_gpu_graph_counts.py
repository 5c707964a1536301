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


def _align(ctx, A, B, T0):
    T, c, st = ctx.align_submaps(A, B, T0)
    return [T, c, st["n_used"]]


def _multistart(ctx, A, B, T0):
    T, c, st = ctx.align_multistart(A, B, T0, n_starts=2)
    return [T, c, st["n_used"]]


def _batch(ctx, A, B, T0):
    T, c, st = ctx.align_batch([(A, B, T0), (B, B, np.eye(4))], 1)
    return [T, c, st[0]["n_used"]]


def _prepared(ctx, A, B, T0):
    S = ctx.align_prepare([(A, B, T0)], 1)
    S.launch()
    T, c, st = S.collect()
    S.close()
    return [T, c, st[0]["n_used"]]


def _sums(ctx, A, B, T0):
    return [ctx.normal_equations(A, B, T0)]


def _poses(ctx, A, B, T0):
    x, st = ctx.pgo_solve([A, B], np.array([[0.0, 0, 0, 0], [0.02, -0.01, 0.01, 0.01]]), [(0, 1)], [])
    return [x, st["cost_init"], st["cost_final"]]


@pytest.mark.parametrize("call", [_align, _multistart, _batch, _prepared, _sums, _poses])
@pytest.mark.parametrize("between", [False, True])  # an eager frame between the replays
def test_alignment_behind_a_replay_with_more_blocks(cv, call, between):
    """A field that a running replay is making, with more blocks than the replay before
    it made: every alignment call sees all of it (bit for bit the eager result)."""
    import torch
    w = sg.tiny()
    fr = w.frames(0, 12)
    full, few = torch.from_numpy(fr).cuda(), torch.from_numpy(fr).cuda()
    few[:, 30:] = 0.0  # the first rows alone
    T0 = np.eye(4)
    T0[:3, 3] = [0.02, -0.01, 0.01]

    def maps(ctx):
        A, B = ctx.submap_create(), ctx.submap_create()
        ctx.integrate_depth_batch(B, full[:6], w.cam.K, w.poses[:6])
        ctx.update_esdf(B)
        assert len(ctx.export_points(B)) > 1000
        return A, B

    kw = dict(block_capacity=1 << 15, w_reg=1.0, **KW)
    ctx = cv.Context(**kw)
    A, B = maps(ctx)
    ctx.integrate_depth_batch(A, full, w.cam.K, w.poses[:12])
    ctx.update_esdf(A)
    most = ctx.submap_info(A)["n_blocks"]
    want = call(ctx, A, B, T0)
    ctx.close()

    ctx = cv.Context(**kw)
    A, B = maps(ctx)
    buf = few.clone()
    ctx.graph_begin()
    ctx.submap_reset(A)
    ctx.integrate_depth_batch(A, buf, w.cam.K, w.poses[:12])
    ctx.update_esdf(A)
    g = ctx.graph_end()
    g.launch()
    assert 0 < ctx.submap_info(A)["n_blocks"] < most - 100
    if between:
        ctx.integrate_depth(A, few[0], w.cam.K, w.poses[0])
    buf.copy_(full)
    ctx.sync()
    busy = _busy()
    g.launch()
    got = call(ctx, A, B, T0)
    assert ctx.submap_info(A)["n_blocks"] == most
    for a, b in zip(got, want):
        assert np.array_equal(a, b)
    del busy
    g.close()
    ctx.close()
