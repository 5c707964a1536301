"""map_sequence whose ESDF passes ride in the next chunk's integration launches,
against the same calls one after another, bit for bit, for each launch that takes them
along or leaves them: frames that might overflow the pool (blocks ordered first),
batches, column segments from the tuning (partial updates), per-line envelopes and
timed kernels (which keep the second stream), and a sequence that overflows."""
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


def _in_order(ctx, s, dev, K, poses, every):
    F = dev.shape[0]
    for f0 in range(0, F, every):
        f1 = min(F, f0 + every)
        if f1 - f0 == 1:
            ctx.integrate_depth(s, dev[f0], K, poses[f0])
        else:
            ctx.integrate_depth_batch(s, dev[f0:f1], K, poses[f0:f1])
        ctx.update_esdf(s)


def _same(a, b):
    for k in ("keys", "D", "W"):
        assert np.array_equal(a[k], b[k]), k
    assert np.array_equal(a["phi"], b["phi"], equal_nan=True)


@pytest.mark.parametrize("every", [1, 2, 7])
@pytest.mark.parametrize("path", ["flags", "tight", "segments", "envelopes", "timed", "fp16 tight"])
def test_sequence_equals_calls_in_order(cv, path, every):
    import torch
    w = sg.tiny()
    fr = w.frames()
    dev = torch.from_numpy(fr).cuda()
    base = dict(voxel_size=0.05, trunc_vox=4, max_range=5.0, d_max=2.0, block_capacity=1 << 17)
    if "fp16" in path:
        base["precision"] = cv.FP16
    ref = cv.Context(**base)
    a = ref.submap_create()
    _in_order(ref, a, dev, w.cam.K, w.poses, every)
    ea = ref.export_blocks(a)
    ref.close()
    if "tight" in path:
        base["block_capacity"] = len(ea["keys"])
    ctx = cv.Context(**base)
    if path == "segments":
        ctx.set_tuning(edt_col_seg=4)
    if path == "envelopes":
        ctx.set_tuning(edt_y_env_min_cols=1, edt_z_env_min_cols=1)
    if path == "timed":
        ctx.timing_enable(["probe", "edt_y"])
    b = ctx.submap_create()
    print("sequence", path, every, flush=True)
    for _ in range(2):  # the second finds buffers of their size and an old ESDF
        ctx.submap_reset(b)
        ctx.map_sequence(b, dev, w.cam.K, w.poses, esdf_every=every)
        _same(ea, ctx.export_blocks(b))
    ctx.close()


def test_overflowing_sequence_keeps_the_last_update(cv):
    """A sequence that overflows at some frame reports it; the blocks and the ESDF
    are those of the frames before."""
    import torch
    w = sg.tiny()
    fr = w.frames()
    dev = torch.from_numpy(fr).cuda()
    base = dict(voxel_size=0.05, trunc_vox=4, max_range=5.0, d_max=2.0)
    big = cv.Context(block_capacity=1 << 17, **base)
    a = big.submap_create()
    n = []
    for f in range(w.n_frames):
        big.integrate_depth(a, dev[f], w.cam.K, w.poses[f])
        n.append(big.submap_info(a)["n_blocks"])
    k = next(i for i in range(1, len(n)) if n[i] > n[0])
    big.submap_reset(a)
    _in_order(big, a, dev[:k], w.cam.K, w.poses[:k], 1)
    ea = big.export_blocks(a)
    ctx = cv.Context(block_capacity=n[k] - 1, **base)
    b = ctx.submap_create()
    print("overflow at frame", k, flush=True)
    with pytest.raises(cv.CovoxError) as e:
        ctx.map_sequence(b, dev, w.cam.K, w.poses, esdf_every=1)
    assert e.value.code == cv.EPOOL_FULL
    _same(ea, ctx.export_blocks(b))
    big.close()
    ctx.close()
