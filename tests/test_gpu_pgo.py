"""GPU parity of the submap pose-graph optimisation (Eq. 1, Sec. III-F
backend) through the C ABI against the oracle's dense Levenberg-Marquardt:
the same iterations and accepted steps, poses within 1e-7 (m, rad).  The
GPU solves each step by preconditioned CG to a relative residual of 1e-12,
the oracle by Cholesky; registration normal equations come from the GPU's
alignment kernel and the oracle's own, which agree to rounding."""
import math

import numpy as np
import pytest

import oracle as orc
from oracle import pgo
import scenegen as sg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cv():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_21149_amd as cv
    return cv


def _chain(N, seed):
    rng = np.random.default_rng(seed)
    x_true = np.zeros((N, 4))
    for k in range(1, N):
        step = np.r_[rng.uniform(1, 2), rng.uniform(-0.5, 0.5), rng.uniform(-0.1, 0.1), rng.uniform(-0.4, 0.4)]
        x_true[k, :3] = x_true[k - 1, :3] + pgo.rz(x_true[k - 1, 3]) @ step[:3]
        x_true[k, 3] = x_true[k - 1, 3] + step[3]
    return x_true, rng


def _rel(xi, xj):
    T = np.linalg.inv(pgo.pose_matrix(xi)) @ pgo.pose_matrix(xj)
    return np.r_[T[:3, 3], math.atan2(T[1, 0], T[0, 0])]


def _compare(xg, sg_, xo, so):
    assert sg_["iterations"] == so["iterations"] and sg_["accepted"] == so["accepted"]
    d = xg - xo
    d[:, 3] = [pgo.wrap(a) for a in d[:, 3]]
    assert np.abs(d).max() <= 1e-7, np.abs(d).max()
    assert abs(sg_["cost_final"] - so["cost_final"]) <= 1e-9 * max(1.0, so["cost_final"])


def test_odometry_and_loop_graph_matches_oracle(cv):
    """Eight poses, noisy odometry and three loop closures, no registration."""
    N = 8
    x_true, rng = _chain(N, 11)
    facs = []
    for k in range(N - 1):
        z = _rel(x_true[k], x_true[k + 1]) + np.r_[rng.normal(scale=0.05, size=3), rng.normal(scale=0.01)]
        facs.append(dict(i=k, j=k + 1, z=z, sigma=[0.05, 0.05, 0.05, 0.01]))
    for (i, j) in ((0, 5), (2, 7), (1, 6)):
        z = _rel(x_true[i], x_true[j]) + np.r_[rng.normal(scale=0.02, size=3), rng.normal(scale=0.005)]
        facs.append(dict(i=i, j=j, z=z, sigma=[0.02, 0.02, 0.02, 0.005]))
    x0 = x_true.copy()
    x0[1:, :3] += rng.normal(scale=0.4, size=(N - 1, 3))
    x0[1:, 3] += rng.normal(scale=0.1, size=N - 1)
    ctx = cv.Context(block_capacity=64)
    subs = [ctx.submap_create() for _ in range(N)]
    xg, sg_ = ctx.pgo_solve(subs, x0, [], facs, max_iter=30)
    xo, so = pgo.solve([], [], x0, [], facs, max_iter=30)
    _compare(xg, sg_, xo, so)
    assert sg_["cost_final"] < 1e-3 * sg_["cost_init"]
    ctx.close()


def test_registration_graph_matches_oracle(cv):
    """The tiny room cut into four submaps of five frames (each frame twice,
    the world frame as submap frame: the true poses are all zero), started
    up to 4 cm / 1.5 deg off, with odometry factors and every ordered
    registration pair."""
    import torch
    w = sg.tiny()
    fr = w.frames()
    dev = torch.from_numpy(fr).cuda()
    ctx = cv.Context(voxel_size=0.05, trunc_vox=4, max_range=5.0, d_max=2.0, block_capacity=8192)
    N = 4
    subs = [ctx.submap_create() for _ in range(N)]
    refs = [orc.Submap(orc.Params()) for _ in range(N)]
    for f in range(20):
        k = f // 5
        for _ in range(2):
            ctx.integrate_depth(subs[k], dev[f], w.cam.K, w.poses[f])
            refs[k].integrate(fr[f], w.cam.K, w.poses[f])
    for s, r in zip(subs, refs):
        ctx.update_esdf(s)
        r.update_esdf()
    pts = [r.iso_points() for r in refs]
    rng = np.random.default_rng(5)
    x0 = np.zeros((N, 4))
    x0[1:, :3] = rng.uniform(-0.03, 0.03, size=(N - 1, 3))
    x0[1:, 3] = np.radians(rng.uniform(-1.5, 1.5, size=N - 1))
    facs = [dict(i=k, j=k + 1, z=[0.0, 0.0, 0.0, 0.0], sigma=[0.2, 0.2, 0.2, 0.05]) for k in range(N - 1)]
    pairs = [(i, j) for i in range(N) for j in range(N) if i != j]
    xg, sg_ = ctx.pgo_solve(subs, x0, pairs, facs, sigma_reg=0.05, max_iter=15)
    xo, so = pgo.solve(refs, pts, x0, pairs, facs, sigma_reg=0.05, max_iter=15)
    _compare(xg, sg_, xo, so)
    assert sg_["accepted"] > 0 and sg_["cost_final"] < 0.1 * sg_["cost_init"]
    ctx.close()


def test_pgo_rejects_bad_input(cv):
    import torch
    ctx = cv.Context(block_capacity=4096)
    subs = [ctx.submap_create() for _ in range(3)]
    x0 = np.zeros((3, 4))
    good = dict(i=0, j=1, z=[1, 0, 0, 0], sigma=[1, 1, 1, 1])
    for bad in (dict(good, j=3), dict(good, j=0), dict(good, sigma=[1, 0, 1, 1])):
        with pytest.raises(cv.CovoxError):
            ctx.pgo_solve(subs, x0, [], [bad])
    with pytest.raises(cv.CovoxError):
        ctx.pgo_solve(subs, x0, [], [])
    w = sg.tiny(n_frames=1)
    ctx.integrate_depth(subs[0], torch.from_numpy(w.frame(0)).cuda(), w.cam.K, w.poses[0])
    with pytest.raises(cv.CovoxError):  # ESDF of submap 0 not updated after integration
        ctx.pgo_solve(subs, x0, [(0, 1)], [good])
    ctx.close()


@pytest.mark.parametrize("N", [2, 17, 18, 65, 66, 90])
def test_solver_sizes_match_oracle(cv, N):
    """Chains with loop closures at the sizes where the solver's form changes:
    one wave (up to 16 free poses), one workgroup with the matrix in LDS (up to
    64), the matrix in memory beyond."""
    x_true, rng = _chain(N, 100 + N)
    facs = []
    edges = [(k, k + 1) for k in range(N - 1)] + [(k, k + 9) for k in range(0, N - 9, 4)]
    for i, j in edges:
        z = _rel(x_true[i], x_true[j]) + np.r_[rng.normal(scale=0.02, size=3), rng.normal(scale=0.005)]
        facs.append(dict(i=i, j=j, z=z, sigma=[0.05, 0.05, 0.05, 0.01]))
    x0 = x_true.copy()
    x0[1:, :3] += rng.normal(scale=0.1, size=(N - 1, 3))
    x0[1:, 3] += rng.normal(scale=0.02, size=N - 1)
    ctx = cv.Context(block_capacity=16)
    subs = [ctx.submap_create() for _ in range(N)]
    xg, sg_ = ctx.pgo_solve(subs, x0, [], facs, max_iter=12)
    xo, so = pgo.solve([], [], x0, [], facs, max_iter=12)
    # CG stops at a residual of 1e-12 of the gradient (the oracle solves densely);
    # a chain of N poses has a condition number of up to about N^2 / sigma^2 ratios
    # of 25, so the steps, and the poses of a few metres, agree to well below 1e-7 m
    assert np.abs(xg - xo).max() <= 1e-7
    assert abs(sg_["cost_final"] - so["cost_final"]) <= 1e-9 * max(1.0, so["cost_final"])
    x1, s1 = ctx.pgo_solve(subs, x0, [], facs, max_iter=0)
    assert np.array_equal(x1, x0) and s1["cost_init"] == s1["cost_final"] and s1["iterations"] == 0
    ctx.close()


@pytest.mark.parametrize("N,reach", [(9, 3), (17, 7), (18, 7), (17, 8), (40, 4), (40, 5)])
def test_rows_of_many_blocks_match_oracle(cv, N, reach):
    """Every pose tied to its `reach` next ones: rows of up to 8 blocks (2 reach + 1
    away from the ends) stay in registers, longer ones are read from LDS, in one wave
    and in a workgroup.  Tolerances as for the solver sizes: the ties only add
    stiffness, so the condition number is not larger."""
    x_true, rng = _chain(N, 300 + N + reach)
    facs = []
    for i in range(N):
        for j in range(i + 1, min(N, i + reach + 1)):
            z = _rel(x_true[i], x_true[j]) + np.r_[rng.normal(scale=0.02, size=3), rng.normal(scale=0.005)]
            facs.append(dict(i=i, j=j, z=z, sigma=[0.05, 0.05, 0.05, 0.01]))
    x0 = x_true.copy()
    x0[1:, :3] += rng.normal(scale=0.1, size=(N - 1, 3))
    x0[1:, 3] += rng.normal(scale=0.02, size=N - 1)
    ctx = cv.Context(block_capacity=16)
    subs = [ctx.submap_create() for _ in range(N)]
    print("rows", N, reach, flush=True)
    xg, sg_ = ctx.pgo_solve(subs, x0, [], facs, max_iter=12)
    xo, so = pgo.solve([], [], x0, [], facs, max_iter=12)
    assert np.abs(xg - xo).max() <= 1e-7
    assert abs(sg_["cost_final"] - so["cost_final"]) <= 1e-9 * max(1.0, so["cost_final"])
    ctx.close()
