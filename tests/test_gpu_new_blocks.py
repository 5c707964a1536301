"""The single-frame path that orders a frame's new blocks from flag bytes (no ordering
kernel of its own): boxes of less than one 16-block read, of a ragged last read, and
of several rounds of reads; a first frame with many new blocks and later ones with a
few, none, or an empty image.  Blocks, order, table homes, counts and box equal those
of the path that a pool without room to spare takes, and the oracle's."""
import numpy as np
import pytest

import oracle as orc
import scenegen as sg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cv():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_21149_amd as cv
    return cv


@pytest.mark.parametrize("vs,far,precision", [
    (0.80, 2.0, "FP32"),  # a box of a few blocks
    (0.25, 5.0, "FP32"),  # some hundred
    (0.10, 5.0, "FP16"),  # one round of reads
    (0.05, 5.0, "FP32"),  # several
    (0.03, 5.0, "FP32"),  # many
])
def test_new_blocks_in_box_order(cv, vs, far, precision):
    import torch
    w = sg.tiny()
    fr = w.frames(0, 8).copy()
    fr[2] = 0.0  # nothing new
    fr[3] = fr[1]
    poses = [w.poses[k] for k in (0, 1, 2, 1, 4, 5, 6, 7)]  # frame 3 repeats frame 1
    dev = torch.from_numpy(fr).cuda()
    kw = dict(voxel_size=vs, trunc_vox=4, max_range=far, d_max=10 * vs, precision=getattr(cv, precision))
    ref = orc.Submap(orc.Params(vs=vs, trunc_vox=4, max_range=far, d_max=10 * vs, fp16=precision == "FP16"))
    for f in range(8):
        ref.integrate(fr[f], w.cam.K, poses[f])
    exp = ref.export()
    need = len(exp["keys"])
    out = []
    # room to spare: new blocks by flags; the blocks needed and no more: ordered first
    for cap in (1 << 17, need):
        print("blocks", vs, need, "of", cap, flush=True)
        ctx = cv.Context(block_capacity=cap, **kw)
        s = ctx.submap_create()
        for f in range(8):
            ctx.integrate_depth(s, dev[f], w.cam.K, poses[f])
        ctx.update_esdf(s)  # over the box of the blocks
        out.append((ctx.export_blocks(s), ctx.submap_info(s)))
        ctx.close()
    (a, ia), (b, ib) = out
    assert need > 0 and ia["n_blocks"] == ib["n_blocks"] == need
    assert ia["n_updates"] == ib["n_updates"]
    for k in ("keys", "D", "W"):
        assert np.array_equal(a[k], b[k]), k
    assert np.array_equal(a["phi"], b["phi"], equal_nan=True)
    assert np.array_equal(a["keys"], exp["keys"])
    assert np.array_equal(a["D"], exp["D"]) and np.array_equal(a["W"], exp["W"])
