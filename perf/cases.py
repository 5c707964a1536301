"""The work that programs built on this library have it do, as measurable cases.

listed() gives the fixed cases and draw() more of the same ranges; prepare() makes what a program
holds before a call (depth frames on the device, mapped submaps, a network), run() is one pass
through the public entry points, work() its unavoidable bytes and operations, and exact() the same
outputs in binary64, written with plain torch from the definitions in include/covox.h.

Scenes are closed-form (a room of spheres and boxes, or sloping ground with mounds and buildings),
seen by a camera on a smooth path with depth-dependent noise and invalid pixels; their sizes, noise
and camera constants are those of the room and outdoor workloads of this repository.
"""
import math

import numpy as np
import torch

import paper_2410_21149_amd as cv

# Room: 8 x 6 x 3 m, 5 cm voxels, 5 m range.  Outdoor: 10 cm voxels, 10 m range.
ENV = {
    "room": dict(vs=0.05, max_range=5.0, d_max=2.0, focal=525.0 / 640.0, noise=0.0012, step=0.04, cell=0.2),
    "outdoor": dict(vs=0.10, max_range=10.0, d_max=3.0, focal=380.0 / 640.0, noise=0.002, step=0.13, cell=1.0),
}
TRUNC = 4
INVALID = 0.1        # share of pixels without a measurement
GRID = 32            # cells per axis of a summary window
CAPACITY = {"room": 131072, "outdoor": 65536}
OUTDOOR_TOL = dict(tol_rho=1e-5, tol_theta=1e-6)
POINTS = 1 << 18     # surface points a program keeps room for
RING = 8             # distinct new frames that a live camera's case cycles through


def listed():
    return [
        # A live camera at low resolution: one frame into the map, ESDF update, the planner's window.
        dict(name="frame_small", kind="frame", env="room", H=120, W=160, warm=12, fp16=False, wavefront=False),
        # The mapping loop of the room workload: an ESDF update after every frame.
        dict(name="sequence_room", kind="sequence", env="room", H=480, W=640, F=60, every=1, fp16=False, inv_depth=False),
        # The same loop at an odd image size, in half-precision storage, sensor-weighted, ESDF every 5 frames.
        dict(name="sequence_fp16_odd", kind="sequence", env="room", H=361, W=487, F=43, every=5, fp16=True, inv_depth=True),
        # An outdoor submap built in one go: 100 frames in batches, then its ESDF.
        dict(name="submap_outdoor", kind="sequence", env="outdoor", H=480, W=640, F=100, every=0, fp16=False, inv_depth=False),
        # Full ESDF of a set of outdoor submaps in one batched update.
        dict(name="esdf_outdoor", kind="esdf", env="outdoor", H=240, W=320, n=16, F=60, seg=0),
        # The raycast integrator on recorded room frames.
        dict(name="raycast_room", kind="raycast", env="room", H=480, W=640, F=6, carve=True),
        # The incremental wavefront ESDF behind a live camera.
        dict(name="wavefront_room", kind="frame", env="room", H=480, W=640, warm=20, fp16=False, wavefront=True),
        # One loop-closure check: a single pair of room submaps.
        dict(name="align_pair", kind="align", env="room", H=240, W=320, subs=2, F=30, n=1, starts=1, lm=False, dof=6),
        # Loop-closure candidates of an outdoor map, eight starts each.
        dict(name="align_outdoor", kind="align", env="outdoor", H=240, W=320, subs=8, F=50, n=64, starts=8, lm=False, dof=6),
        # The proposal network on the pairs of one call.
        dict(name="net_forward", kind="forward", n=64),
        # One training batch of the proposal network.
        dict(name="net_gradients", kind="gradients", n=64),
        # The pose graph over the submaps of a trajectory.
        dict(name="pose_graph", kind="pgo", env="outdoor", H=240, W=320, subs=16, F=40, reach=3),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the ranges the listed ones stand for."""
    kind = rng.choice(["frame", "sequence", "sequence", "esdf", "raycast", "align", "align", "forward", "gradients", "pgo"])
    env = rng.choice(["room", "outdoor"])
    W = _log(rng, 160, 640)
    H = max(90, min(480, int(W * rng.choice([0.5625, 0.75])) + rng.randrange(-3, 4)))
    if kind == "frame":
        return dict(kind=kind, env=env, H=H, W=W, warm=rng.randrange(2, 21), fp16=rng.random() < 0.3,
                    wavefront=rng.random() < 0.3)
    if kind == "sequence":
        F = _log(rng, 5, 60)
        return dict(kind=kind, env=env, H=H, W=W, F=F, every=rng.choice([0, 1, 1, rng.randrange(2, 9)]),
                    fp16=rng.random() < 0.3, inv_depth=rng.random() < 0.3)
    if kind == "esdf":
        return dict(kind=kind, env=env, H=120, W=160 + rng.randrange(0, 9), n=_log(rng, 1, 16), F=rng.randrange(10, 41),
                    seg=rng.choice([0, 0, 8, 32]))
    if kind == "raycast":
        return dict(kind=kind, env="room", H=H, W=W, F=rng.randrange(1, 6), carve=rng.random() < 0.7)
    if kind == "align":
        lm, dof = rng.random() < 0.3, rng.choice([6, 6, 4])
        if rng.random() < 0.5:
            return dict(kind=kind, env=env, H=180, W=240, subs=2, F=rng.randrange(10, 31), n=1, starts=rng.choice([1, 8]),
                        lm=lm, dof=dof)
        return dict(kind=kind, env=env, H=180, W=240, subs=5, F=rng.randrange(15, 31), n=_log(rng, 2, 60),
                    starts=rng.choice([1, 4, 8]), lm=lm, dof=dof)
    if kind == "pgo":
        return dict(kind=kind, env="outdoor", H=120, W=160 + rng.randrange(0, 9), subs=rng.randrange(3, 13),
                    F=rng.randrange(20, 41), reach=rng.randrange(1, 4))
    return dict(kind=kind, n=_log(rng, 1, 64))


# ------------------------------------------------------------------ scenes

def _scene(env, rng):
    """Spheres (n, 4) and boxes (m, 6), float32 on the device."""
    if env == "room":
        sph = [[*rng.uniform([0.6, 0.6, 0.3], [7.4, 5.4, 2.7]), rng.uniform(0.1, 0.45)] for _ in range(20)]
        box = []
        for _ in range(20):
            side = rng.uniform(0.2, 0.9, 3)
            lo = rng.uniform([0.1, 0.1, 0.0], [7.8 - side[0], 5.8 - side[1], 2.3 - side[2]])
            box.append([*lo, *(lo + side)])
        # nothing within half a metre of the camera's path (an ellipse about the centre)
        ring = [(4.0 + 1.0 * math.cos(a), 3.0 + 0.7 * math.sin(a), 1.5) for a in np.linspace(0, 2 * math.pi, 40)]
        sph = [s for s in sph if all(math.dist(s[:3], q) > s[3] + 0.5 for q in ring)]
        box = [b for b in box if all(max(max(b[a] - q[a], q[a] - b[a + 3]) for a in range(3)) > 0.4 for q in ring)]
    else:
        sph, box = [], []
        for _ in range(60):  # mounds: spheres sunk into the ground
            r, h = rng.uniform(2.0, 9.0), rng.uniform(0.3, 1.3)
            sph.append([rng.uniform(-12, 75), rng.uniform(-16, 16), h - r, r])
        for _ in range(50):  # rubble
            r = rng.uniform(0.25, 0.9)
            sph.append([rng.uniform(-8, 70), rng.uniform(-12, 12), rng.uniform(0.0, 0.4) * r, r])
        for _ in range(18):  # buildings and walls on both sides of the path
            side = rng.uniform([1.0, 0.4, 1.0], [7.0, 4.0, 4.0])
            y = rng.choice([-1, 1]) * rng.uniform(4.5, 9.0)
            x = rng.uniform(-5, 70)
            box.append([x, y - side[1] / 2, -0.5, x + side[0], y + side[1] / 2, side[2]])
    dev = dict(dtype=torch.float32, device="cuda")
    return torch.tensor(np.array(sph).reshape(-1, 4), **dev), torch.tensor(np.array(box).reshape(-1, 6), **dev)


def _pose(pos, yaw, pitch):
    """T_world_cam of a camera at pos (x right, y down, z forward)."""
    f = np.array([math.cos(pitch) * math.cos(yaw), math.cos(pitch) * math.sin(yaw), math.sin(pitch)])
    x = np.cross(f, [0.0, 0.0, 1.0])
    x /= np.linalg.norm(x)
    T = np.eye(4)
    T[:3, 0], T[:3, 1], T[:3, 2], T[:3, 3] = x, np.cross(f, x), f, pos
    return T


def _path(env, F, first, phase):
    """Poses first .. first + F - 1 of the camera's path."""
    out = []
    for k in range(first, first + F):
        s = k * ENV[env]["step"]
        if env == "room":
            a = phase + s
            pos = [4.0 + 1.0 * math.cos(a), 3.0 + 0.7 * math.sin(a), 1.5 + 0.2 * math.sin(1.3 * s + phase)]
            out.append(_pose(pos, a + 0.9 + 0.26 * math.sin(3.1 * s + phase), 0.17 * math.sin(4.2 * s)))
        else:
            pos = [s, 1.2 * math.sin(0.15 * s + phase), 3.2 + 0.7 * math.sin(0.21 * s + phase)]
            out.append(_pose(pos, 0.35 * math.sin(0.17 * s + phase), -0.5))
    return np.array(out)


def _camera(case):
    H, W = case["H"], case["W"]
    f = ENV[case["env"]]["focal"] * W
    return np.array([f, f, (W - 1) / 2.0, (H - 1) / 2.0], np.float32)


def _render(case, scene, poses, gen):
    """Depth frames (F, H, W) float32 on the device, 0 where there is no measurement."""
    e, K, H, W = ENV[case["env"]], _camera(case), case["H"], case["W"]
    sph, box = scene
    u = (torch.arange(W, device="cuda", dtype=torch.float32) - float(K[2])) / float(K[0])
    v = (torch.arange(H, device="cuda", dtype=torch.float32) - float(K[3])) / float(K[1])
    cam = torch.stack([u[None, :].expand(H, W), v[:, None].expand(H, W), torch.ones(H, W, device="cuda")], -1)
    out = torch.empty((len(poses), H, W), device="cuda")
    per = max(1, (4 << 20) // (H * W))
    for f0 in range(0, len(poses), per):
        P = torch.tensor(poses[f0:f0 + per], dtype=torch.float32, device="cuda")
        d = [sum(cam[None, ..., c] * P[:, r, c, None, None] for c in range(3)) for r in range(3)]
        o = [P[:, r, 3, None, None] for r in range(3)]
        d = [torch.where(x.abs() < 1e-9, torch.full_like(x, 1e-9), x) for x in d]
        if case["env"] == "room":
            t = torch.full_like(d[0], 1e9)
            for a, (lo, hi) in enumerate(((0.0, 8.0), (0.0, 6.0), (0.0, 3.0))):
                t = torch.minimum(t, torch.where(d[a] > 0, (hi - o[a]) / d[a], (lo - o[a]) / d[a]))
        else:
            t = torch.where(d[2] < 0, -o[2] / d[2], torch.full_like(d[2], 1e9))
        dd = d[0] * d[0] + d[1] * d[1] + d[2] * d[2]
        for s in sph:
            q = [o[a] - s[a] for a in range(3)]
            b = q[0] * d[0] + q[1] * d[1] + q[2] * d[2]
            disc = b * b - dd * (q[0] * q[0] + q[1] * q[1] + q[2] * q[2] - s[3] * s[3])
            r = (-b - disc.clamp_min(0).sqrt()) / dd
            t = torch.where((disc > 0) & (r > 0), torch.minimum(t, r), t)
        inv = [1.0 / x for x in d]
        for bx in box:
            lo = [(bx[a] - o[a]) * inv[a] for a in range(3)]
            hi = [(bx[a + 3] - o[a]) * inv[a] for a in range(3)]
            near = torch.maximum(torch.maximum(torch.minimum(lo[0], hi[0]), torch.minimum(lo[1], hi[1])), torch.minimum(lo[2], hi[2]))
            far = torch.minimum(torch.minimum(torch.maximum(lo[0], hi[0]), torch.maximum(lo[1], hi[1])), torch.maximum(lo[2], hi[2]))
            t = torch.where((near < far) & (near > 0), torch.minimum(t, near), t)
        t = t + e["noise"] * t * t * torch.randn(t.shape, device="cuda", generator=gen)
        bad = (torch.rand(t.shape, device="cuda", generator=gen) < INVALID) | (t > e["max_range"]) | (t <= 0)
        out[f0:f0 + per] = torch.where(bad, torch.zeros_like(t), t)
    return out


def _gravity(T):
    """A submap pose: position and yaw of the camera pose T, no roll or pitch."""
    yaw = math.atan2(T[1, 2], T[0, 2])
    G = np.eye(4)
    G[:2, :2] = [[math.cos(yaw), -math.sin(yaw)], [math.sin(yaw), math.cos(yaw)]]
    G[:3, 3] = T[:3, 3]
    return G


def _submaps(case):
    n = case.get("n", 1) if case["kind"] == "esdf" else case.get("subs", 1)
    return n


def _frames_of(case):
    return case["warm"] + RING if case["kind"] == "frame" else case["F"]


def _inputs(case, seed):
    """Per submap: (T_world_submap, poses, frames); made from the seed alone."""
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    scene = _scene(case["env"], rng)
    phase = rng.uniform(0, 2 * math.pi)
    F = _frames_of(case)
    apart = F if case["kind"] == "esdf" else max(1, F // 3)  # aligned submaps overlap
    if case["env"] == "outdoor":
        apart = min(apart, 400 // max(1, _submaps(case)))
    out = []
    for k in range(_submaps(case)):
        poses = _path(case["env"], F, k * apart, phase)
        out.append((_gravity(poses[0]), poses, _render(case, scene, poses, gen)))
    return out


def _params(case):
    e = ENV[case["env"]]
    p = dict(voxel_size=e["vs"], trunc_vox=TRUNC, max_range=e["max_range"], d_max=e["d_max"],
             block_capacity=CAPACITY[case["env"]])
    if case["kind"] in ("esdf", "align", "pgo", "raycast"):
        p["block_capacity"] = 16384
    if case["env"] == "outdoor":
        p.update(OUTDOOR_TOL)
    if case.get("fp16"):
        p["precision"] = cv.FP16
    if case.get("inv_depth"):
        # weights 1 / d^2 of distant surfaces are below the default weight of a registration endpoint
        p.update(weight_mode=cv.WEIGHT_INV_DEPTH2, w_reg=0.2)
    if case.get("wavefront"):
        p["esdf_mode"] = cv.ESDF_WAVEFRONT
    if case["kind"] == "raycast":
        p.update(integrator=cv.RAYCAST, ray_carve=int(case["carve"]))
    if case.get("lm"):
        p["align_solver"] = cv.LEVENBERG_MARQUARDT
    p["align_dof"] = case.get("dof", 6)
    return p


# ------------------------------------------------------------------- cases

def _window_pose(case, T_ws, poses):
    """The window looks ahead of the last camera pose: T_submap_grid."""
    G = np.eye(4)
    ahead = 2.0 if case["env"] == "room" else 4.0
    P = poses[-1]
    G[:3, 3] = (np.linalg.inv(T_ws) @ np.append(P[:3, 3] + ahead * P[:3, 2], 1.0))[:3]
    return G


def _priors(case, inputs, seed):
    """(a, b, T_init) of the alignment problems: ground truth moved as odometry drift moves it."""
    rng = np.random.default_rng(seed + 77)
    n_sub = len(inputs)
    cand = [(a, b) for a in range(n_sub) for b in range(n_sub) if a != b and abs(a - b) <= 2]
    # the tilt of a 4-DoF prior is exact; one start stands for a refined prior, eight for a coarse one
    coarse = case["starts"] > 1 and case["env"] == "outdoor"
    t, yaw = (0.5, math.radians(10)) if coarse else (0.08, math.radians(2))
    out = []
    for k in range(case["n"]):
        a, b = cand[k % len(cand)]
        gt = np.linalg.inv(inputs[a][0]) @ inputs[b][0]
        w = rng.uniform(-yaw, yaw)
        D = np.eye(4)
        D[:2, :2] = [[math.cos(w), -math.sin(w)], [math.sin(w), math.cos(w)]]
        D[:3, 3] = rng.uniform(-t, t, 3) * [1, 1, 0.3]
        out.append((a, b, gt @ D))
    return out


def _graph(case, inputs, seed):
    """Initial poses, registration pairs and odometry factors of the pose graph."""
    rng = np.random.default_rng(seed + 78)
    n = len(inputs)
    x = np.array([[*T[:3, 3], math.atan2(T[1, 0], T[0, 0])] for T, _, _ in inputs])

    def rel(i, j):
        c, s = math.cos(x[i, 3]), math.sin(x[i, 3])
        d = x[j, :3] - x[i, :3]
        return np.array([c * d[0] + s * d[1], -s * d[0] + c * d[1], d[2], x[j, 3] - x[i, 3]])

    sigma = np.array([0.05, 0.05, 0.05, 0.01])
    odo = [dict(i=i, j=i + 1, z=(rel(i, i + 1) + sigma * rng.standard_normal(4)).tolist(), sigma=sigma.tolist()) for i in range(n - 1)]
    x0 = x.copy()
    for f in odo:  # dead reckoning
        i, z = f["i"], f["z"]
        c, s = math.cos(x0[i, 3]), math.sin(x0[i, 3])
        x0[i + 1] = [x0[i, 0] + c * z[0] - s * z[1], x0[i, 1] + s * z[0] + c * z[1], x0[i, 2] + z[2], x0[i, 3] + z[3]]
    pairs = [(i, j) for i in range(n) for j in range(i + 1, min(n, i + 1 + case["reach"]))]
    return x0, pairs, odo


def _net_input(n, seed):
    """Network inputs as the summaries give them: smooth clamped distances with an observed mask per
    channel pair, and regression targets (correction within +-3 m, any yaw)."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    low = torch.rand((n, 4, 6, 6, 6), device="cuda", generator=gen) * 2 - 1
    f = torch.nn.functional.interpolate(low, size=(GRID, GRID, GRID), mode="trilinear", align_corners=True)
    x = torch.empty((n, GRID, GRID, GRID, 4), device="cuda")
    for s in range(2):
        m = (f[:, 2 * s + 1] > -0.25).float()
        x[..., 2 * s] = (2.0 * f[:, 2 * s]).clamp(-1, 1) * m
        x[..., 2 * s + 1] = m
    r = torch.rand((n, 4), device="cuda", generator=gen) * 2 - 1
    y = torch.stack([3 * r[:, 0], 3 * r[:, 1], 0.5 * r[:, 2], (math.pi * r[:, 3]).cos(), (math.pi * r[:, 3]).sin()], 1)
    return x.contiguous(), y.contiguous()


def _net_weights(seed):
    """Trained-size weights: He-uniform kernels and small biases."""
    rng = np.random.default_rng(seed + 5)
    out = []
    for cin, cout in ((4, 16), (16, 32), (32, 64), (64, 64)):
        out += [rng.uniform(-1, 1, cout * 27 * cin) * math.sqrt(6.0 / (27 * cin)), rng.uniform(0.0, 0.1, cout)]
    out += [rng.uniform(-1, 1, 5 * 64) * math.sqrt(6.0 / 64), rng.uniform(-0.1, 0.1, 5)]
    return np.concatenate(out).astype(np.float32)


def prepare(case, seed):
    st = dict(case=case)
    kind = case["kind"]
    if kind in ("forward", "gradients"):
        st["ctx"] = cv.Context(block_capacity=64)
        st["net"] = cv.Net(st["ctx"], seed=1)
        st["net"].set_params(_net_weights(seed))
        st["x"], st["y"] = _net_input(case["n"], seed)
        return st
    inputs = _inputs(case, seed)
    torch.cuda.synchronize()  # the frames are complete before another stream reads them
    st["stream"] = torch.cuda.Stream()
    ctx = st["ctx"] = cv.Context(stream=st["stream"], **_params(case))
    K = st["K"] = _camera(case)
    subs = st["subs"] = [ctx.submap_create(T) for T, _, _ in inputs]
    st["windows"] = [_window_pose(case, T, P) for T, P, _ in inputs]
    st["out"] = torch.zeros((len(subs), GRID, GRID, GRID, 4), device="cuda")
    st["inputs"] = inputs
    if kind in ("sequence", "raycast"):
        st["points"], st["n_points"] = np.zeros((POINTS, 3), np.float32), 0
    if kind == "frame":
        T, P, D = inputs[0]
        w = case["warm"]
        ctx.integrate_depth_batch(subs[0], D[:w], K, P[:w])
        ctx.update_esdf(subs[0])
        st["next"] = 0
    elif kind in ("esdf", "align", "pgo"):
        for s, (_, P, D) in zip(subs, inputs):
            ctx.integrate_depth_batch(s, D, K, P)
        if kind == "esdf":
            ctx.set_tuning(edt_col_seg=case["seg"], esdf_full_recompute=1)
        else:
            ctx.update_esdf_batch(subs)
        if kind == "align":
            st["pairs"] = [(subs[a], subs[b], T) for a, b, T in _priors(case, inputs, seed)]
        if kind == "pgo":
            st["graph"] = _graph(case, inputs, seed)
    ctx.sync()
    torch.cuda.synchronize()
    return st


def _windows(st):
    cell = ENV[st["case"]["env"]]["cell"]
    st["ctx"].summaries([(s, G, cell, st["out"][k], 0) for k, (s, G) in enumerate(zip(st["subs"], st["windows"]))])
    return st["out"]


def _surface(st):
    """The submap's surface points in the program's buffer, zero beyond them."""
    p, buf = st["ctx"].export_points(st["subs"][0]), st["points"]
    buf[:len(p)] = p
    buf[len(p):st["n_points"]] = 0
    st["n_points"] = len(p)
    return buf


def run(st):
    """One pass.  Maps come back as what programs read from them: the planner's window of the ESDF
    (value and mask per cell) and, for a finished submap, its surface points."""
    case, ctx = st["case"], st["ctx"]
    kind = case["kind"]
    if kind == "forward":
        return st["net"].forward(st["x"])
    if kind == "gradients":
        loss, g = st["net"].gradients(st["x"], st["y"])
        return {"loss": loss, "grad": g}
    subs, K = st["subs"], st["K"]
    if kind == "frame":
        _, P, D = st["inputs"][0]
        f = case["warm"] + st["next"] % RING
        st["next"] += 1
        ctx.integrate_depth(subs[0], D[f], K, P[f])
        ctx.update_esdf(subs[0])
        return {"window": _windows(st)}
    if kind == "sequence":
        _, P, D = st["inputs"][0]
        ctx.submap_reset(subs[0])
        ctx.map_sequence(subs[0], D, K, P, esdf_every=case["every"])
        return {"window": _windows(st), "points": _surface(st)}
    if kind == "raycast":
        _, P, D = st["inputs"][0]
        ctx.submap_reset(subs[0])
        ctx.integrate_depth_batch(subs[0], D, K, P)
        ctx.update_esdf(subs[0])
        return {"window": _windows(st), "points": _surface(st)}
    if kind == "esdf":
        ctx.update_esdf_batch(subs)
        return {"window": _windows(st)}
    if kind == "align":
        if case["n"] == 1 and case["starts"] == 1:
            A, B, T0 = st["pairs"][0]
            T, cost, stats = ctx.align_submaps(A, B, T0)
            T, cost, stats = T[None], np.array([cost]), [stats]
        else:
            T, cost, stats = ctx.align_batch(st["pairs"], case["starts"])
        whole = np.array([[s["n_points"], s["n_used"], s["iterations"], s["status"], s["best_start"]] for s in stats])
        return {"T": T, "cost": cost, "stats": whole}
    x0, pairs, odo = st["graph"]
    x, stats = ctx.pgo_solve(subs, x0, pairs, odo)
    return {"x": x, "cost": np.array([stats["cost_init"], stats["cost_final"]])}


# -------------------------------------------------------------------- work

def work(case):
    """Bytes and operations a pass cannot do without.  Voxel, block and point counts are those that
    the generated scenes give on average."""
    kind = case["kind"]
    if kind in ("forward", "gradients"):
        n = case["n"]
        convs = ((4, 16, 32), (16, 32, 16), (32, 64, 8), (64, 64, 4))
        fwd = sum(2 * 27 * ci * co * o ** 3 for ci, co, o in convs) * n
        if kind == "forward":
            return {"bytes": n * GRID ** 3 * 16 + 4 * 181941 + 20 * n, "flops": fwd}
        return {"bytes": n * GRID ** 3 * 16 + 8 * 181941 + 20 * n, "flops": 3 * fwd - 2 * 27 * 4 * 16 * GRID ** 3 * n}
    e = ENV[case["env"]]
    vs, px = e["vs"], case["H"] * case["W"]
    s_dw = 4 if case.get("fp16") else 8
    # voxels that a frame observes, blocks of the first frame and new blocks of each later one
    upd, first, more = (6.5e4, 380, 16) if case["env"] == "room" else (1.1e5, 850, 12)
    blocks = first + more * _frames_of(case)
    per_frame = 4 * px + 2 * s_dw * upd
    esdf = (s_dw + 4) * 512
    win = GRID ** 3 * 16
    if kind == "frame":
        return {"bytes": per_frame + esdf * blocks + win, "flops": 40 * upd}
    if kind in ("sequence", "raycast"):
        F = case["F"]
        every = case.get("every", 0)
        updates = 1 if every <= 0 else -(-F // every)
        ray = 16 * upd if kind == "raycast" else 0
        grown = sum(first + more * min(F, (k + 1) * max(every, 1)) for k in range(updates)) if every > 0 else blocks
        steps = px * (60 if kind == "raycast" else 0)
        return {"bytes": F * (per_frame + ray) + esdf * grown + s_dw * 512 * blocks + win, "flops": F * (40 * upd + 30 * steps)}
    if kind == "esdf":
        return {"bytes": case["n"] * (esdf * blocks + win), "flops": case["n"] * blocks * 512 * 100.0}
    # fields and registration points read once; 150 operations a point and evaluation
    pts, evals = (1.5e4 if case["env"] == "room" else 2.5e4), 20
    if kind == "align":
        evals *= case["n"] * case["starts"]
    else:
        evals *= sum(min(case["reach"], case["subs"] - 1 - i) for i in range(case["subs"]))
    return {"bytes": case["subs"] * (12 * pts + 2048 * blocks), "flops": 150 * pts * evals}


# ------------------------------------------------------- binary64 reference

def _dense(case, T_ws, poses, frames):
    """Dense voxel box of a submap that holds everything its frames can observe: (lo, dim, vs)."""
    vs, H, W = ENV[case["env"]]["vs"], case["H"], case["W"]
    K = _camera(case).astype(np.float64)
    u = (torch.arange(W, device="cuda", dtype=torch.float64) - K[2]) / K[0]
    v = (torch.arange(H, device="cuda", dtype=torch.float64) - K[3]) / K[1]
    lo, hi = np.full(3, np.inf), np.full(3, -np.inf)
    for P, d in zip(poses, frames):
        T = np.linalg.inv(T_ws) @ P
        z = d.double()
        cam = torch.stack([(z * u[None, :]).reshape(-1), (z * v[:, None]).reshape(-1), z.reshape(-1)])
        p = torch.tensor(T[:3, :3], device="cuda") @ cam + torch.tensor(T[:3, 3:], device="cuda")
        lo = np.minimum(lo, p.amin(1).cpu().numpy())
        hi = np.maximum(hi, p.amax(1).cpu().numpy())
    m = TRUNC + 4
    lo = np.floor(lo / vs).astype(int) - m
    dim = np.ceil(hi / vs).astype(int) + m - lo
    return lo, dim, vs


def _centres(lo, dim, vs):
    ax = [(torch.arange(int(n), device="cuda", dtype=torch.float64) + float(o) + 0.5) * vs for o, n in zip(lo, dim)]
    return torch.meshgrid(*ax, indexing="ij")


def _tsdf(case, T_ws, poses, frames, box):
    """D and W of the dense box by projection mapping."""
    e, K = ENV[case["env"]], _camera(case).astype(np.float64)
    H, W, tau = case["H"], case["W"], TRUNC * box[2]
    X = _centres(*box)
    D = torch.zeros(X[0].shape, dtype=torch.float64, device="cuda")
    Wt = torch.zeros_like(D)
    for P, depth in zip(poses, frames):
        T = np.linalg.inv(P) @ T_ws
        p = [T[r, 0] * X[0] + T[r, 1] * X[1] + T[r, 2] * X[2] + T[r, 3] for r in range(3)]
        front = p[2] > 0
        z = torch.where(front, p[2], torch.ones_like(p[2]))
        c = torch.floor(K[0] * p[0] / z + K[2] + 0.5)
        r = torch.floor(K[1] * p[1] / z + K[3] + 0.5)
        ok = front & (c >= 0) & (c < W) & (r >= 0) & (r < H)
        d = depth.double().reshape(-1)[torch.where(ok, r * W + c, torch.zeros_like(c)).long()]
        sdf = d - p[2]
        ok &= (d > 0) & (d <= e["max_range"]) & (sdf >= -tau)
        w = torch.where(ok, 1.0 / (d * d) if case.get("inv_depth") else torch.ones_like(d), torch.zeros_like(d))
        Wn = Wt + w
        D = torch.where(ok, (D * Wt + sdf.clamp_max(tau) * w) / Wn, D)
        Wt = torch.where(ok, Wn, Wt)
    return D, Wt


def _tsdf_raycast(case, T_ws, poses, frames, box):
    """D and W of the dense box by raycasting: every voxel a ray crosses, summed per frame."""
    e, K = ENV[case["env"]], _camera(case).astype(np.float64)
    lo, dim, vs = box
    tau = TRUNC * vs
    D = torch.zeros(tuple(int(n) for n in dim), dtype=torch.float64, device="cuda").reshape(-1)
    Wt = torch.zeros_like(D)
    lo_t = torch.tensor(lo, device="cuda").long()[:, None]
    col = torch.arange(case["W"], device="cuda", dtype=torch.float64)
    row = torch.arange(case["H"], device="cuda", dtype=torch.float64)
    for P, depth in zip(poses, frames):
        T = np.linalg.inv(T_ws) @ P
        z = depth.double()
        ok = (z > 0) & (z <= e["max_range"])
        q = torch.stack([((col[None, :] - K[2]) * z / K[0])[ok], ((row[:, None] - K[3]) * z / K[1])[ok], z[ok]])
        d = torch.tensor(T[:3, :3], device="cuda") @ q
        r = d.norm(dim=0)
        u = d / r
        o = torch.tensor(T[:3, 3:], device="cuda")
        s0 = torch.zeros_like(r) if case["carve"] else (r - tau).clamp_min(0)
        i = torch.floor((o + s0 * u) / vs).long()
        step = torch.sign(u).long()
        sw, stw = torch.zeros_like(D), torch.zeros_like(D)
        alive = torch.ones_like(r, dtype=torch.bool)
        at, ts = [], []
        while bool(alive.any()):
            c = (i.double() + 0.5) * vs
            sdf = r - ((c - o) * u).sum(0)
            hit = alive & (sdf >= -tau)
            j = (i - lo_t)[:, hit]
            a = (j[0] * int(dim[1]) + j[1]) * int(dim[2]) + j[2]
            at.append(a)
            ts.append(sdf[hit].clamp_max(tau))
            s = torch.where(step != 0, ((i + (step > 0).long()).double() * vs - o) / u, torch.full_like(u, math.inf))
            sm, ax = s.min(0)
            alive &= sm < r + tau
            i = i + torch.nn.functional.one_hot(ax, 3).T * step * alive
        a, order = torch.cat(at).sort()
        run = torch.cat(ts)[order].cumsum(0)
        a, n = a.unique_consecutive(return_counts=True)
        end = run[n.cumsum(0) - 1]
        sw[a] = n.double()
        stw[a] = torch.diff(end, prepend=end.new_zeros(1))
        ok = sw > 0
        Wn = Wt + sw
        D = torch.where(ok, (D * Wt + stw) / Wn, D)
        Wt = torch.where(ok, Wn, Wt)
    shape = tuple(int(n) for n in dim)
    return D.reshape(shape), Wt.reshape(shape)


def _esdf(case, D, W, vs):
    """phi of the dense box (NaN where unobserved)."""
    d_max, tau = ENV[case["env"]]["d_max"], TRUNC * vs
    R = round(d_max / vs)
    obs = W > 0
    k = torch.where(obs & (D.abs() <= vs), 0.0, 1e9).float()
    for a in range(3):
        n = k.shape[a]
        best = k.clone()
        for s in range(1, min(R, n - 1) + 1):
            best.narrow(a, s, n - s).copy_(torch.minimum(best.narrow(a, s, n - s), k.narrow(a, 0, n - s) + s * s))
            best.narrow(a, 0, n - s).copy_(torch.minimum(best.narrow(a, 0, n - s), k.narrow(a, s, n - s) + s * s))
        k = best
    far = torch.where(k <= R * R, (vs * k.double().sqrt()).clamp_max(d_max), torch.full_like(D, d_max))
    phi = torch.where(D > 0, far, -far)
    phi = torch.where(D.abs() < tau * (1 - 2.0 ** -10), D, phi)
    return torch.where(obs, phi, torch.full_like(phi, math.nan))


def _field(case, inp, frames=None):
    T_ws, poses, depth = inp
    if frames is not None:
        poses, depth = poses[:frames], depth[:frames]
    box = _dense(case, T_ws, poses, depth)
    D, W = (_tsdf_raycast if case["kind"] == "raycast" else _tsdf)(case, T_ws, poses, depth, box)
    return box, D, W, _esdf(case, D, W, box[2])


def _corners(box, phi, q):
    """The 8 corner values and cell fractions of points q (3, n); good: all corners observed."""
    lo, dim, vs = box
    g = q / vs - 0.5
    f = torch.floor(g)
    fr, j = g - f, f.long() - torch.tensor(lo, device="cuda").long()[:, None]
    n = torch.tensor([int(x) for x in dim], device="cuda")[:, None]
    inside = ((j >= 0) & (j + 1 < n)).all(0)
    j = torch.where(inside, j, torch.zeros_like(j))
    c = [phi[j[0] + (k & 1), j[1] + ((k >> 1) & 1), j[2] + (k >> 2)] for k in range(8)]
    good = inside & ~torch.stack(c).isnan().any(0)
    return [torch.where(good, x, torch.zeros_like(x)) for x in c], fr, good


def _trilinear(c, f):
    """Value and gradient (per cell) of the trilinear patch."""
    x, y, z = f
    c00, c10, c01, c11 = (c[k] * (1 - x) + c[k + 1] * x for k in (0, 2, 4, 6))
    c0, c1 = c00 * (1 - y) + c10 * y, c01 * (1 - y) + c11 * y
    dx = ((c[1] - c[0]) * (1 - y) + (c[3] - c[2]) * y) * (1 - z) + ((c[5] - c[4]) * (1 - y) + (c[7] - c[6]) * y) * z
    return c0 * (1 - z) + c1 * z, torch.stack([dx, (c10 - c00) * (1 - z) + (c11 - c01) * z, c1 - c0])


def _exact_window(case, inp, field):
    box, _, _, phi = field
    e = ENV[case["env"]]
    c = (torch.arange(GRID, device="cuda", dtype=torch.float64) + 0.5 - GRID / 2) * e["cell"]
    zz, yy, xx = torch.meshgrid(c, c, c, indexing="ij")
    G = _window_pose(case, inp[0], inp[1])
    q = torch.stack([xx.reshape(-1), yy.reshape(-1), zz.reshape(-1)]) + torch.tensor(G[:3, 3:], device="cuda")
    cs, f, good = _corners(box, phi, q)
    val, _ = _trilinear(cs, f)
    out = torch.zeros((GRID ** 3, 4), dtype=torch.float64, device="cuda")
    out[:, 0] = torch.where(good, (val / e["d_max"]).clamp(-1, 1), torch.zeros_like(val))
    out[:, 1] = good.double()
    return out.reshape(GRID, GRID, GRID, 4)


def _points(case, field, w_reg=2.0):
    """Registration points (3, n): zero crossings along the edges of the dense box."""
    (lo, dim, vs), D, W, _ = field
    ok = (W >= w_reg) & (D.abs() < TRUNC * vs * (1 - 2.0 ** -10))
    X = torch.stack(_centres(lo, dim, vs))
    out = []
    for a in range(3):
        n = D.shape[a] - 1
        p, q = D.narrow(a, 0, n), D.narrow(a, 1, n)
        m = ok.narrow(a, 0, n) & ok.narrow(a, 1, n) & ((p < 0) != (q < 0))
        pts = X.narrow(a + 1, 0, n)[:, m].clone()
        pts[a] += vs * (p / (p - q))[m]
        out.append(pts)
    return torch.cat(out, 1)


def _exp(xi):
    """SE(3) exponential of (rho, theta)."""
    M = torch.zeros((4, 4), dtype=torch.float64)
    r, w = xi[:3], xi[3:]
    M[:3, :3] = torch.tensor([[0, -w[2], w[1]], [w[2], 0, -w[0]], [-w[1], w[0], 0]])
    M[:3, 3] = r
    return torch.linalg.matrix_exp(M)


def _residuals(box, phi, q):
    c, f, good = _corners(box, phi, q)
    r, g = _trilinear(c, f)
    return r[good], g[:, good] / box[2], good


def _exact_align(case, inputs, priors):
    """One Gauss-Newton solve per pair (one start), to convergence or 30 updates."""
    fields = [_field(case, i) for i in inputs]
    sel = [0, 1, 2, 5] if case["dof"] == 4 else list(range(6))
    tr, tt = (OUTDOOR_TOL["tol_rho"], OUTDOOR_TOL["tol_theta"]) if case["env"] == "outdoor" else (1e-7, 1e-8)
    Ts, costs = [], []
    for a, b, T0 in priors:
        box, phi, p = fields[a][0], fields[a][3], _points(case, fields[b])
        T, it, done = torch.tensor(T0, dtype=torch.float64), 0, False
        while True:
            Td = T.cuda()
            q = Td[:3, :3] @ p + Td[:3, 3:]
            r, g, good = _residuals(box, phi, q)
            if done or it >= 30:
                break
            J = torch.cat([g, torch.linalg.cross(q[:, good], g, dim=0)])[sel]
            delta = torch.zeros(6, dtype=torch.float64)
            delta[sel] = torch.linalg.solve((J @ J.T).cpu(), -(J @ r).cpu())
            T = _exp(delta) @ T
            it += 1
            done = bool(delta[:3].norm() < tr and delta[3:].norm() < tt)
        Ts.append(T.numpy())
        costs.append(float((r * r).mean()))
    return {"T": np.array(Ts), "cost": np.array(costs), "stats": None}


def _rz(a):
    c, s = math.cos(a), math.sin(a)
    return torch.tensor([[c, -s, 0], [s, c, 0], [0, 0, 1]], dtype=torch.float64, device="cuda")


def _exact_graph(case, inputs, graph):
    """The pose graph by Levenberg-Marquardt with dense normal equations."""
    x0, pairs, odo = graph
    fields = [_field(case, i) for i in inputs]
    pts = [_points(case, f) for f in fields]
    n, w_reg = len(inputs), 1.0 / 0.05 ** 2
    turn = torch.tensor([[0, -1, 0], [1, 0, 0], [0, 0, 0]], dtype=torch.float64, device="cuda")

    def linearise(x):
        H, g, F = torch.zeros((4 * n, 4 * n), dtype=torch.float64), torch.zeros(4 * n, dtype=torch.float64), 0.0
        X = torch.tensor(x, device="cuda")
        for i, j in pairs:
            Ri, Rj, d = _rz(x[i, 3]), _rz(x[j, 3]), (X[j, :3] - X[i, :3])[:, None]
            m = Rj @ pts[j] + d
            r, gr, good = _residuals(fields[i][0], fields[i][3], Ri.T @ m)
            gw = Ri @ gr
            J = torch.cat([-gw, (gr * ((turn @ Ri).T @ m[:, good])).sum(0)[None],
                           gw, (gw * (turn @ Rj @ pts[j][:, good])).sum(0)[None]])
            at = [4 * i + k for k in range(4)] + [4 * j + k for k in range(4)]
            H[np.ix_(at, at)] += w_reg * (J @ J.T).cpu()
            g[at] += w_reg * (J @ r).cpu()
            F += w_reg * float((r * r).sum())
        for f in odo:
            i, j, z, w = f["i"], f["j"], torch.tensor(f["z"]).double(), 1.0 / torch.tensor(f["sigma"]).double() ** 2

            def err(v):
                def back(a, t):
                    c, s = torch.cos(a), torch.sin(a)
                    return torch.stack([c * t[0] + s * t[1], -s * t[0] + c * t[1], t[2]])
                t = back(z[3], back(v[3], v[4:7] - v[:3]) - z[:3])
                y = v[7] - v[3] - z[3]
                return torch.cat([t, torch.atan2(torch.sin(y), torch.cos(y))[None]])
            v = torch.tensor(np.concatenate([x[i], x[j]]))
            e, J = err(v), torch.autograd.functional.jacobian(err, v).T
            at = [4 * i + k for k in range(4)] + [4 * j + k for k in range(4)]
            H[np.ix_(at, at)] += J @ (w[:, None] * J.T)
            g[at] += J @ (w * e)
            F += float((w * e * e).sum())
        return H[4:, 4:], g[4:], F

    x, mu, nu = np.array(x0), 1e-4, 2.0
    H, g, F = linearise(x)
    F0 = F
    for _ in range(20):
        delta = torch.linalg.solve(H + mu * torch.diag(H.diagonal()), -g)
        if float(delta.abs().max()) < 1e-8:
            break
        xn = x.copy()
        xn[1:] += delta.numpy().reshape(-1, 4)
        Hn, gn, Fn = linearise(xn)
        rho = (F - Fn) / float(-(2 * delta @ g + delta @ H @ delta))
        if rho > 0:
            x, H, g, F = xn, Hn, gn, Fn
            mu, nu = mu * max(1 / 3, 1 - (2 * rho - 1) ** 3), 2.0
        else:
            mu, nu = mu * nu, 2 * nu
    return {"x": x, "cost": np.array([F0, F])}


def _exact_net(case, seed):
    x, y = _net_input(case["n"], seed)
    w = torch.tensor(_net_weights(seed), dtype=torch.float64, device="cuda", requires_grad=True)
    a, at = x.double(), 0
    for cin, cout, stride in ((4, 16, 1), (16, 32, 2), (32, 64, 2), (64, 64, 2)):
        k = w[at:at + cout * 27 * cin].reshape(cout, 27, cin)
        b = w[at + cout * 27 * cin:at + cout * 27 * cin + cout]
        at += cout * 27 * cin + cout
        p = torch.nn.functional.pad(a, (0, 0, 1, 1, 1, 1, 1, 1))
        o = a.shape[1] // stride
        acc = b.expand(a.shape[0], o, o, o, cout)
        for t in range(27):
            z, yy, xx = t // 9, t // 3 % 3, t % 3
            acc = acc + p[:, z:z + stride * o:stride, yy:yy + stride * o:stride, xx:xx + stride * o:stride] @ k[:, t].T
        a = acc.relu()
    out = a.mean((1, 2, 3)) @ w[at:at + 320].reshape(5, 64).T + w[at + 320:]
    if case["kind"] == "forward":
        return out.detach()
    scale = torch.tensor([1 / 9.0] * 3 + [1.0] * 2, dtype=torch.float64, device="cuda")
    loss = ((out - y.double()) ** 2 * scale).sum() / case["n"]
    loss.backward()
    return {"loss": float(loss), "grad": w.grad.cpu().numpy()}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("forward", "gradients"):
        return _exact_net(case, seed)
    if kind == "align" and (case["starts"] > 1 or case["lm"]):
        return None  # hundreds of dense solves, with a choice among starts at near-equal costs
    inputs = _inputs(case, seed)
    if kind == "align":
        return _exact_align(case, inputs, _priors(case, inputs, seed))
    if kind == "pgo":
        return _exact_graph(case, inputs, _graph(case, inputs, seed))
    n = case["warm"] + 1 if kind == "frame" else None
    win = torch.stack([_exact_window(case, i, _field(case, i, n)) for i in inputs])
    # the points' number follows the last bits of D: no value of their own in 64 bits
    return {"window": win, "points": None} if kind in ("sequence", "raycast") else {"window": win}
