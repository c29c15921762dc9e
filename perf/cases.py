"""The work a user of this framework has it do, as cases that can be timed and compared.

A case is a dict of plain values.  Its "kind" says which entry points it goes
through, its other values are sizes and options:

  track   one camera stream (Tracker)
          form "pair":   one live frame against a prepared reference: its
                         pyramid and its track, waited for
          form "window": a keyframe window: the reference update from a depth
                         map, then `frames` frames in one window track
          form "frames": the same window frame by frame, enqueued
          form "tween":  the tween-window schedule: two anchors, then frames
                         each waited for
  batch   `streams` streams together (BatchTracker)
          form "window": as above, every stream
          form "pair":   one frame of every stream from a given start;
                         sizes 0: every stream its own resolution and map size
          form "learned": one frame of every stream from the network's proposal
  train   a training step of the learned initialiser (Cnn)
  select  map-point selection on a device image (select_points_noalloc)

Tracks return the poses, the mean costs and the statuses.  The tracker's state
and sums are FP32, widened to doubles only by the result structure, so poses and
costs are returned as FP32.  Iteration, sample and visible-point counts are
diagnostics of a run: a step within rounding of the convergence threshold, or a
point within rounding of the image border, moves them by one.

Inputs: a seeded textured scene of three planes seen from a smooth seeded
motion, with pixel noise, rendered on the GPU.
"""
import math
import os

import numpy as np
import torch

import paper_2607_16897_amd as dpt

HUBER_K, STEP_EPS, Z_MIN, MIN_POINTS, MAX_ITERS, MARGIN = 9.0, 1e-5, 1e-3, 10, 10, 8
LAUNCH = {"auto": (dpt.LAUNCH_AUTO, 256), "pairs": (dpt.LAUNCH_COOP_PAIRS, 128)}


def listed():
    track = dict(kind="track", form="window", width=752, height=480, points=2000, levels=4, frames=9, option="fp32",
                 patch=0, gauss=False, launch="pairs")
    batch = dict(kind="batch", form="window", streams=64, width=752, height=480, points=2000, levels=4, frames=9,
                 option="fp32")
    return [
        # one live frame on a small map: the smallest call, where latency and launches count
        dict(track, name="live_640x480_500", form="pair", width=640, height=480, points=500, levels=3, frames=1,
             launch="auto"),
        # the same on frames of odd sizes and a large map, default launch
        dict(track, name="live_1241x719_7001", form="pair", width=1241, height=719, points=7001, frames=1, launch="auto"),
        # the benchmark's keyframe window: reference update and nine tween frames of one stream
        dict(track, name="window_752x480_2000"),
        # the constant-H track on an odd frame size and map, default launch
        dict(track, name="fixed_h_641x479_1111", width=641, height=479, points=1111, option="fixed_h", launch="auto"),
        # the precision stress: 1280x720, 16000 points, FP16 template cache
        dict(track, name="mixed_1280x720_16000", width=1280, height=720, points=16000, option="mixed", launch="auto"),
        # the paper's shape: floating-point Gaussian pyramid, six levels, 7x7 patches, frame by frame
        dict(track, name="paper_752x480_7x7", form="frames", levels=6, patch=7, gauss=True, launch="auto"),
        # the schedule a SLAM front end runs: anchors from the indirect side, each direct frame waited for
        dict(track, name="tween_752x480_2000", form="tween", launch="auto"),
        # a server's batch: 64 sequences of the benchmark's shape, one keyframe window each
        dict(batch, name="batch64_window"),
        # a server's batch of cameras of all resolutions and map sizes, one frame each
        dict(batch, name="batch64_mixed_sizes", form="pair", width=0, height=0, points=0, levels=3, frames=1),
        # one frame of 64 streams started from the learned proposal
        dict(batch, name="batch64_learned", form="learned", frames=1),
        # a training step of the initialiser at its training batch
        dict(kind="train", name="train_256", batch=256),
        # point selection on a large image of odd size
        dict(kind="select", name="select_2047x1535", width=2047, height=1535, points=16000, margin=8),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    pick = rng.choice(["pair", "window", "window", "frames", "tween", "batch", "batch", "learned", "train", "select"])
    if pick == "train":
        return dict(kind="train", batch=_log(rng, 5, 256))
    if pick == "select":
        w, h = _log(rng, 320, 2047), _log(rng, 240, 1535)
        return dict(kind="select", width=w, height=h, points=_log(rng, 300, 16000), margin=rng.randint(1, 16))
    if pick == "learned":  # the network reads the 94 x 60 level of 752 x 480
        return dict(kind="batch", form="learned", streams=_log(rng, 2, 64), width=752, height=480,
                    points=_log(rng, 300, 2500), levels=4, frames=1, option=rng.choice(["fp32", "mixed"]))
    w, h = rng.choice([(640, 480), (752, 480), (1280, 720), (0, 0)])
    if w == 0:
        w, h = rng.randint(320, 1280), rng.randint(240, 720)
    case = dict(width=w, height=h, points=_log(rng, 300, 8000), levels=rng.randint(3, 4), frames=1)
    if pick == "batch":
        case.update(kind="batch", form=rng.choice(["window", "pair"]), streams=_log(rng, 2, 48),
                    option=rng.choice(["fp32", "fp32", "mixed", "fixed_h"]))
        case["points"] = min(case["points"], 64 * 2000 // case["streams"])
        if case["form"] == "window":
            case["frames"] = rng.randint(2, 9)
        return case
    case.update(kind="track", form=pick, option=rng.choice(["fp32", "fp32", "mixed", "fixed_h"]), patch=0, gauss=False,
                launch=rng.choice(["auto", "pairs"]))
    if pick != "pair":
        case["frames"] = rng.randint(2, 9)
    if pick in ("frames", "window") and rng.random() < 0.5:  # the paper's patches
        case.update(patch=rng.choice([3, 5, 7]), gauss=pick == "frames", points=min(case["points"], 3000),
                    levels=4 if pick == "window" else rng.randint(3, 5), option=rng.choice(["fp32", "fixed_h"]),
                    launch="auto")
    if case["launch"] == "pairs":
        case["points"] = min(case["points"], 4000)
    return case


# ---------------------------------------------------------------- inputs


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _rotation(w):
    """exp of the rotation vector w (numpy, FP64)."""
    th = float(np.linalg.norm(w))
    W = np.array([[0, -w[2], w[1]], [w[2], 0, -w[0]], [-w[1], w[0], 0]])
    if th < 1e-8:
        return np.eye(3) + W
    return np.eye(3) + math.sin(th) / th * W + (1 - math.cos(th)) / th ** 2 * (W @ W)


def _pose(R, t):
    T = np.eye(4)
    T[:3, :3], T[:3, 3] = R, t
    return T


def _motion(rng, n):
    """n + 2 camera poses of a smooth motion: about 2.5 mm and 0.1 degrees a frame,
    the first before the reference, the second the reference's."""
    T = _pose(_rotation(rng.uniform(-0.1, 0.1, 3)), rng.uniform(-0.2, 0.2, 3))
    w, v = rng.normal(0.0, 0.001, 3), rng.normal(0.0, 0.0014, 3)
    out = []
    for _ in range(n + 2):
        out.append(T)
        w, v = w + rng.normal(0.0, 0.00008, 3), v + rng.normal(0.0, 0.0001, 3)
        T = _pose(_rotation(w), v) @ T
    return out


def _offset(rng, deg, metres):
    """A pose at most `deg` degrees and `metres` away."""
    a, d = rng.normal(size=3), rng.normal(size=3)
    return _pose(_rotation(a / np.linalg.norm(a) * math.radians(rng.uniform(0, deg))),
                 d / np.linalg.norm(d) * rng.uniform(0, metres))


def _camera(w, h):
    f = 458.0 / 752.0 * w if w == 752 else 460.0 / 640.0 * w
    return dpt.Camera(w, h, f, f, 0.49 * w, 0.51 * h)


def _render(cam, poses, seed, n_depths=1):
    """Frames [F, H, W] uint8 of the seeded scene at the world-to-camera poses, and
    the depth maps of the first n_depths: the planes y = -1, z = 3 and x = 2 with
    one continuous 3-D texture of three octaves, and pixel noise of sigma 2."""
    dev = _device()
    g = torch.Generator(device=dev).manual_seed(int(seed))
    n = 32
    vol = torch.rand((n, n, n), generator=g, device=dev)
    vol = torch.cat([vol, vol[:1]], 0)
    vol = torch.cat([vol, vol[:, :1]], 1)
    vol = torch.cat([vol, vol[:, :, :1]], 2).reshape(-1)
    x = (torch.arange(cam.width, device=dev, dtype=torch.float64) - cam.cx) / cam.fx
    y = (torch.arange(cam.height, device=dev, dtype=torch.float64) - cam.cy) / cam.fy
    y, x = torch.meshgrid(y, x, indexing="ij")
    rays = torch.stack([x, y, torch.ones_like(x)], -1)
    out = torch.empty((len(poses), cam.height, cam.width), dtype=torch.uint8, device=dev)
    depths = []
    for k, T in enumerate(poses):
        T = torch.as_tensor(T, dtype=torch.float64, device=dev)
        d, c = rays @ T[:3, :3], -(T[:3, 3] @ T[:3, :3])
        z = torch.full_like(x, 1e9)
        for axis, at in ((1, -1.0), (2, 3.0), (0, 2.0)):
            lam = (at - c[axis]) / d[..., axis]
            z = torch.where((lam > 0) & (lam < z), lam, z)
        P = (c + z[..., None] * d).float()
        v = torch.full((cam.height, cam.width), 128.0, device=dev)
        for cell, amp in ((0.025, 40.0), (0.11, 70.0), (0.47, 90.0)):
            q = P / cell + 1000.0 * n
            i = q.floor()
            f = q - i
            f = f * f * (3.0 - 2.0 * f)
            j = i.long() % n
            a = (j[..., 0] * (n + 1) + j[..., 1]) * (n + 1) + j[..., 2]
            acc = 0.0
            for o in range(8):
                ox, oy, oz = o >> 2, (o >> 1) & 1, o & 1
                wt = (f[..., 0] if ox else 1 - f[..., 0]) * (f[..., 1] if oy else 1 - f[..., 1]) * \
                    (f[..., 2] if oz else 1 - f[..., 2])
                acc = acc + wt * vol[a + (ox * (n + 1) + oy) * (n + 1) + oz]
            v = v + amp * (acc - 0.5)
        v = v + 2.0 * torch.randn(v.shape, generator=g, device=dev)
        out[k] = v.round().clamp(0, 255).to(torch.uint8)
        if k < n_depths:
            depths.append(z.float())
    return out, depths


def _streams(case, seed):
    """(camera, points) of every stream of a case."""
    if case["width"]:
        return [(_camera(case["width"], case["height"]), case["points"])] * case.get("streams", 1)
    rng = np.random.default_rng([seed, 3])
    sizes = ((640, 480), (752, 480), (1280, 720))
    return [(_camera(*sizes[rng.integers(3)]), int(round(math.exp(rng.uniform(math.log(300), math.log(8000))))))
            for _ in range(case["streams"])]


def _inputs(case, seed):
    """Every stream's poses, frames (the reference first) and reference depth."""
    out = []
    for s, (cam, points) in enumerate(_streams(case, seed)):
        rng = np.random.default_rng([seed, 7, s])
        if case["form"] in ("pair", "learned"):
            T = _pose(_rotation(rng.uniform(-0.1, 0.1, 3)), rng.uniform(-0.2, 0.2, 3))
            deg, metres = (1.0, 0.02) if case["form"] == "pair" else (2.0, 0.04)
            poses, shown = [T, T, _offset(rng, deg, metres) @ T], 1
        else:
            poses = _motion(rng, case["frames"])
            shown = 0 if case["form"] == "tween" else 1
        # the schedule anchors the frame before the reference too
        frames, depths = _render(cam, poses[shown:], seed * 64 + s, 2 - shown)
        out.append(dict(cam=cam, points=points, poses=poses, frames=frames, depth=depths[-1], depth_before=depths[0]))
    return out


def _patch(case):
    p = case.get("patch", 0)
    return dpt.DEFAULT_PATTERN if not p else [(x, y) for y in range(-(p // 2), p // 2 + 1)
                                              for x in range(-(p // 2), p // 2 + 1)]


def _params(case):
    return dpt.make_params(levels=case["levels"], max_iters=MAX_ITERS, huber_k=HUBER_K, step_eps=STEP_EPS, z_min=Z_MIN,
                           min_points=MIN_POINTS, pattern=_patch(case),
                           precision=dpt.PREC_MIXED if case["option"] == "mixed" else dpt.PREC_FP32,
                           fixed_h=case["option"] == "fixed_h", gauss=case.get("gauss", False))


def _network():
    return np.load(os.path.join(os.path.dirname(dpt.__file__), "weights", "initialiser.npy"), allow_pickle=False)


def _train_inputs(case, seed):
    dev = _device()
    g = torch.Generator(device=dev).manual_seed(int(seed))
    B = case["batch"]
    coarse = torch.rand((B, 2, 8, 12), generator=g, device=dev)
    img = torch.nn.functional.interpolate(coarse, size=(60, 94), mode="bilinear") * 200.0 + 28.0
    img = img + 8.0 * torch.randn(img.shape, generator=g, device=dev)
    pairs = img.round().clamp(0, 255).to(torch.uint8).contiguous()
    return pairs, 0.5 * torch.randn((B, 6), generator=g, device=dev)


def prepare(case, seed):
    if case["kind"] == "train":
        net = dpt.Cnn(max_batch=case["batch"])
        net.set_params(_network())
        pairs, targets = _train_inputs(case, seed)
        return dict(case=case, net=net, pairs=pairs, targets=targets)
    if case["kind"] == "select":
        T = _motion(np.random.default_rng([seed, 7, 0]), 0)[1]
        img = _render(_camera(case["width"], case["height"]), [T], seed)[0][0]
        return dict(case=case, img=img, idx=torch.zeros(case["points"], dtype=torch.int32, device=img.device),
                    count=torch.zeros(1, dtype=torch.int32, device=img.device))
    ins = _inputs(case, seed)
    state = dict(case=case, ins=ins)
    if case["kind"] == "track":
        a = ins[0]
        trk = dpt.Tracker(a["cam"], _params(case), max_points=a["points"])
        trk.set_launch_config(*LAUNCH[case["launch"]])
        if case["form"] == "pair":
            trk.build_pyramid(dpt.SLOT_REF, a["frames"][0])
            trk.set_reference_from_depth(a["points"], a["depth"], a["poses"][1], margin=MARGIN)
        if case["form"] == "tween":
            trk.tween_set_policy(max_cost=1e6, max_direct=case["frames"], n_points=a["points"], margin=MARGIN)
        state.update(trk=trk)
        return state
    bt = dpt.BatchTracker([a["cam"] for a in ins], _params(case), [a["points"] for a in ins])
    state.update(bt=bt, before=np.stack([a["poses"][0] for a in ins]), ref=np.stack([a["poses"][1] for a in ins]),
                 points=[a["points"] for a in ins], depths=[a["depth"] for a in ins],
                 refs=[a["frames"][0] for a in ins], curs=[a["frames"][1] for a in ins],
                 windows=[a["frames"][1:] for a in ins])
    if case["form"] != "window":
        bt.build_pyramids(dpt.SLOT_REF, state["refs"])
        bt.set_reference_from_depth_all(state["points"], state["depths"], state["ref"], margin=MARGIN)
    if case["form"] == "learned":
        state["net"] = dpt.Cnn(max_batch=len(ins))
        state["net"].set_params(_network())
    return state


# ---------------------------------------------------------------- one pass


def _results(T, cost, status):
    return dict(pose=np.asarray(T, np.float32).reshape(-1, 4, 4), cost=np.asarray(cost, np.float32).reshape(-1),
                status=np.asarray(status, np.int32).reshape(-1))


def _of_arrays(r):
    return _results(r["T_cw"], r["final_cost"], r["status"])


def run(state):
    case = state["case"]
    if case["kind"] == "train":
        loss = state["net"].train_step(state["pairs"], state["targets"], 1e-4)
        return dict(loss=np.float32(loss), grads=state["net"].get_grads())
    if case["kind"] == "select":
        dpt.select_points_noalloc(state["img"], case["points"], case["margin"], state["idx"], state["count"])
        return dict(idx=state["idx"], count=state["count"])
    if case["kind"] == "batch":
        bt = state["bt"]
        if case["form"] == "window":
            bt.build_pyramids(dpt.SLOT_REF, state["refs"])
            bt.set_reference_from_depth_all(state["points"], state["depths"], state["ref"], margin=MARGIN)
            bt.set_pose_history_all(state["before"], state["ref"])
            bt.track_window_enqueue(state["windows"])
        else:
            bt.build_pyramids(dpt.SLOT_CUR, state["curs"])
            if case["form"] == "learned":
                state["net"].propose(bt)
                bt.track_enqueue(proposed=True)
            else:
                bt.track_enqueue(state["ref"])
        return _of_arrays(bt.synchronize(arrays=True))
    trk, a = state["trk"], state["ins"][0]
    if case["form"] == "pair":
        trk.build_pyramid(dpt.SLOT_CUR, a["frames"][1])
        r = trk.track(a["poses"][1])
        return _results(r["T_cw"], r["final_cost"], r["status"])
    if case["form"] == "tween":
        trk.tween_anchor(a["frames"][0], a["depth_before"], a["poses"][0])
        trk.tween_anchor(a["frames"][1], a["depth"], a["poses"][1])
        got = [trk.tween_frame(f) for f in a["frames"][2:]]
        out = _results([r["track"]["T_cw"] for r in got], [r["track"]["final_cost"] for r in got],
                       [r["track"]["status"] for r in got])
        out["decision"] = np.array([r["decision"] for r in got], np.int32)
        return out
    trk.build_pyramid(dpt.SLOT_REF, a["frames"][0])
    trk.set_reference_from_depth(a["points"], a["depth"], a["poses"][1], margin=MARGIN)
    trk.set_pose_history(a["poses"][0], a["poses"][1])
    if case["form"] == "window":
        trk.track_window_enqueue(a["frames"][1:])
    else:
        for f in a["frames"][1:]:
            trk.build_pyramid(dpt.SLOT_CUR, f)
            trk.track_enqueue()
    return _of_arrays(trk.synchronize(arrays=True))


_CONVS = ((2, 16, 30, 47), (16, 32, 15, 24), (32, 64, 8, 12), (64, 64, 4, 6))  # CI, CO, Ho, Wo


def work(case):
    conv = [2 * ho * wo * co * 9 * ci for ci, co, ho, wo in _CONVS]
    if case["kind"] == "train":
        B = case["batch"]
        return dict(bytes=B * (2 * 60 * 94 + 24) + 4 * 2 * 65000, flops=B * (3 * sum(conv) - conv[0]))
    if case["kind"] == "select":
        return dict(bytes=case["width"] * case["height"] + 4 * case["points"], flops=5 * case["width"] * case["height"])
    K = len(_patch(case))
    total = dict(bytes=0.0, flops=0.0)
    for cam, points in _streams(case, 0):
        frames = case["frames"] + (2 if case["form"] == "tween" else 0 if case["form"] in ("pair", "learned") else 1)
        # frames in, depths of the selected points, results; about four iterations a level and the final
        # cost, 30 operations a sample and 150 a point each
        total["bytes"] += frames * cam.width * cam.height + 4 * points + 200 * case["frames"]
        total["flops"] += case["frames"] * (4 * case["levels"] + 1) * points * (30 * K + 150)
        if case["form"] == "learned":
            total["flops"] += sum(conv)
    return total


# ---------------------------------------------------------------- the same in 64 bits


def _levels(cam, n):
    return [dict(W=cam.width >> l, H=cam.height >> l, fx=cam.fx / 2 ** l, fy=cam.fy / 2 ** l,
                 cx=(cam.cx + 0.5) / 2 ** l - 0.5, cy=(cam.cy + 0.5) / 2 ** l - 0.5) for l in range(n)]


def _pyramid(img, n, gauss):
    """n levels: 2x2 means of bytes rounded half up, or the [1 3 3 1] / 8 blur of real values."""
    out = [img.double()]
    for _ in range(n - 1):
        p = out[-1]
        h, w = p.shape[0] // 2, p.shape[1] // 2
        if gauss:
            rows = torch.arange(h, device=p.device)[:, None] * 2 - 1 + torch.arange(4, device=p.device)
            cols = torch.arange(w, device=p.device)[:, None] * 2 - 1 + torch.arange(4, device=p.device)
            wt = torch.tensor([1.0, 3.0, 3.0, 1.0], dtype=torch.float64, device=p.device) / 8
            p = (p[rows.clamp(0, p.shape[0] - 1)] * wt[:, None]).sum(1)
            p = (p[:, cols.clamp(0, p.shape[1] - 1)] * wt).sum(2)
        else:
            q = p[:2 * h, :2 * w]
            p = torch.floor((q[::2, ::2] + q[1::2, ::2] + q[::2, 1::2] + q[1::2, 1::2] + 2) / 4)
        out.append(p)
    return out


def _select(img, n, m):
    """The n pixels of the largest squared central differences, ties to the smaller index, ascending."""
    p = img.long()
    h, w = p.shape
    dx, dy = p[m:h - m, m + 1:w - m + 1] - p[m:h - m, m - 1:w - m - 1], p[m + 1:h - m + 1, m:w - m] - p[m - 1:h - m - 1, m:w - m]
    score = (dx * dx + dy * dy).reshape(-1)
    best = torch.sort(score, descending=True, stable=True)[1][:n].sort()[0]
    wc = w - 2 * m
    return (best // wc + m) * w + best % wc + m


def _bilinear(img, x, y):
    i, j = x.floor(), y.floor()
    a, c = x - i, y - j
    at = lambda dx, dy: img[(j + dy).long(), (i + dx).long()]  # noqa: E731
    val = lambda f: (1 - a) * (1 - c) * f(0, 0) + a * (1 - c) * f(1, 0) + (1 - a) * c * f(0, 1) + a * c * f(1, 1)  # noqa: E731
    return val, at


def _project(g, X, pat):
    """Pixel of the points X [n, 3] and whether the whole pattern can be sampled there."""
    u, v = g["fx"] * X[:, 0] / X[:, 2] + g["cx"], g["fy"] * X[:, 1] / X[:, 2] + g["cy"]
    lo, hi = pat.min(0)[0], pat.max(0)[0]
    ok = (X[:, 2] > Z_MIN) & (u + lo[0] >= 1) & (u + hi[0] < g["W"] - 2) & (v + lo[1] >= 1) & (v + hi[1] < g["H"] - 2)
    return u, v, ok


def _exp(xi):
    """SE(3) exponential of (rotation, translation), numpy."""
    w, v = xi[:3], xi[3:]
    th = float(np.linalg.norm(w))
    W = np.array([[0, -w[2], w[1]], [w[2], 0, -w[0]], [-w[1], w[0], 0]])
    if th < 1e-5:
        b, c = 0.5 - th * th / 24, 1 / 6 - th * th / 120
    else:
        b, c = 2 * math.sin(th / 2) ** 2 / th ** 2, (th - math.sin(th)) / th ** 3
    return _pose(_rotation(w), (np.eye(3) + b * W + c * (W @ W)) @ v)


def _orthonormal(T):
    u, _, vt = np.linalg.svd(T[:3, :3])
    return _pose(u @ vt, T[:3, 3])


class _Reference:
    """The inverse-compositional reference and its coarse-to-fine Gauss-Newton track, in 64 bits."""

    def __init__(self, case, a, img, depth, T_rw):
        dev = img.device
        self.case, self.T_rw, self.lv = case, T_rw, _levels(a["cam"], case["levels"])
        self.pat = torch.tensor(_patch(case), dtype=torch.float64, device=dev)
        cam, idx = a["cam"], _select(img, a["points"], MARGIN)
        y, x = torch.div(idx, cam.width, rounding_mode="floor").double(), (idx % cam.width).double()
        z = depth.reshape(-1)[idx].double()
        R, t = (torch.as_tensor(q, device=dev) for q in (T_rw[:3, :3], T_rw[:3, 3]))
        P = (torch.stack([(x - cam.cx) / cam.fx * z, (y - cam.cy) / cam.fy * z, z], 1) - t) @ R
        self.x0 = P.float().double() @ R.T + t  # map points are FP32
        self.cache = []
        for g, p in zip(self.lv, _pyramid(img, case["levels"], case.get("gauss", False))):
            u, v, ok = _project(g, self.x0, self.pat)
            X = self.x0[ok]
            sx, sy = u[ok][:, None] + self.pat[:, 0], v[ok][:, None] + self.pat[:, 1]
            val, at = _bilinear(p, sx, sy)
            gx = val(lambda i, j: (at(i + 1, j) - at(i - 1, j)) / 2)
            gy = val(lambda i, j: (at(i, j + 1) - at(i, j - 1)) / 2)
            iz, xp, yp = 1 / X[:, 2], X[:, 0] / X[:, 2], X[:, 1] / X[:, 2]
            o = torch.zeros_like(iz)
            ju = g["fx"] * torch.stack([-xp * yp, 1 + xp * xp, -yp, iz, o, -xp * iz], 1)
            jv = g["fy"] * torch.stack([-1 - yp * yp, xp * yp, xp, o, iz, -yp * iz], 1)
            J = gx[..., None] * ju[:, None] + gy[..., None] * jv[:, None]  # [n, K, 6]
            H = torch.einsum("nki,nkj->ij", J, J) if case["option"] == "fixed_h" else None
            self.cache.append((X, val(at), J, H))

    def _residuals(self, l, img, T):
        X, I0, J, _ = self.cache[l]
        M = torch.as_tensor(T, device=X.device)
        u, v, ok = _project(self.lv[l], X @ M[:3, :3].T + M[:3, 3], self.pat)
        val, at = _bilinear(img, u[ok][:, None] + self.pat[:, 0], v[ok][:, None] + self.pat[:, 1])
        return I0[ok] - val(at), J[ok], int(ok.sum())

    def track(self, img, T_cw):
        robust = self.case["option"] != "fixed_h"
        pyr = _pyramid(img, self.case["levels"], self.case.get("gauss", False))
        T, status = _orthonormal(T_cw @ np.linalg.inv(self.T_rw)), 0
        for l in reversed(range(self.case["levels"])):
            for it in range(MAX_ITERS):
                r, J, n = self._residuals(l, pyr[l], T)
                if n < MIN_POINTS:
                    status = 2
                    break
                w = (HUBER_K / r.abs().clamp_min(1e-300)).clamp_max(1.0) if robust else torch.ones_like(r)
                J = J.reshape(-1, 6)
                H = self.cache[l][3] if not robust else J.T @ (J * w.reshape(-1, 1))
                b = -(J.T @ (w * r).reshape(-1))
                d = np.linalg.solve(H.cpu().numpy(), b.cpu().numpy())
                T = T @ _exp(-d)
                if np.abs(d).max() < STEP_EPS:
                    break
            else:
                status = 1 if l == 0 else status
            if status == 2:
                break
        r, _, n = self._residuals(0, pyr[0], T)
        rho = 0.5 * r * r
        if robust:
            rho = torch.where(r.abs() > HUBER_K, HUBER_K * (r.abs() - 0.5 * HUBER_K), rho)
        return _orthonormal(T) @ self.T_rw, float(rho.mean()) if n else 0.0, status


def _forward(p, pairs):
    """The network's outputs for byte pairs [B, 2, 60, 94] and parameter tensors p, real arithmetic."""
    h = (pairs.double() - 128.0) / 64.0
    for l in range(4):
        w = p["w%d" % (l + 1)]
        ho, wo = _CONVS[l][2:]
        cols = torch.nn.functional.unfold(h, 3, padding=1, stride=2)
        h = torch.relu(w.reshape(w.shape[0], -1) @ cols + p["b%d" % (l + 1)][:, None]).reshape(len(h), -1, ho, wo)
    h = torch.relu(h.mean((2, 3)) @ p["fw1"].T + p["fb1"])
    return h @ p["fw2"].T + p["fb2"]


def _tensors(flat, dev):
    return {k: torch.as_tensor(np.ascontiguousarray(v)).double().to(dev).requires_grad_(True)
            for k, v in dpt.cnn_unflatten(flat).items()}


def exact(case, seed):
    if case["kind"] == "train":
        pairs, targets = _train_inputs(case, seed)
        p = _tensors(_network(), pairs.device)
        loss = ((_forward(p, pairs) - targets.double()) ** 2).mean()
        loss.backward()
        return dict(loss=loss.item(), grads=torch.cat([p[k].grad.reshape(-1) for k, _ in dpt.CNN_SHAPES]))
    if case["kind"] == "select":
        return None  # whole numbers
    poses, costs = [], []
    for a in _inputs(case, seed):
        first = 2 if case["form"] == "tween" else 1
        ref = _Reference(case, a, a["frames"][first - 1], a["depth"], a["poses"][1])
        older, newer = a["poses"][0], a["poses"][1]
        start = newer
        if case["form"] == "learned":
            pair = torch.stack([_pyramid(a["frames"][k], 4, False)[3] for k in (0, 1)])[None]
            with torch.no_grad():
                xi = _forward(_tensors(_network(), pair.device), pair)[0].cpu().numpy()
            start = _exp(xi * dpt.CNN_TWIST_SCALE) @ newer
        for f in a["frames"][first:]:
            if case["form"] not in ("pair", "learned"):
                start = _orthonormal(newer @ np.linalg.inv(older) @ newer)
            T, cost, _ = ref.track(f, start)
            older, newer = newer, T
            poses.append(T)
            costs.append(cost)
    n, F = len(_streams(case, seed)), case["frames"]
    order = [s * F + f for f in range(F) for s in range(n)]  # results come frame by frame, each of all streams
    return dict(pose=np.stack([poses[i] for i in order]), cost=np.array([costs[i] for i in order]), status=None,
                **(dict(decision=None) if case["form"] == "tween" else {}))
