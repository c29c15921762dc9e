"""The constant-velocity start from a pose history that is off SO(3): poses with
entries rounded to two decimals, as text files hold them.  The predicted start
P1 P0^-1 P1 comes back on SO(3) by two Newton-Schulz steps, so its cost is that
of the same start formed in FP64, projected with two steps, and given.  One step
leaves about 3/8 of the square of the rounding's ~1e-2, a few hundredths of a
pixel at these focal lengths, and a cost off by more than the bound below (FP32
sums of a few thousand terms, a few 1e-6)."""
import numpy as np
import pytest
from scipy.spatial.transform import Rotation

import synth

pytestmark = pytest.mark.gpu

CAM = synth.Camera(640, 480, 900.0, 900.0, 320.0, 240.0)


def _pose(rotvec_deg, t):
    T = np.eye(4)
    T[:3, :3] = Rotation.from_rotvec(np.deg2rad(rotvec_deg)).as_matrix()
    T[:3, 3] = t
    return T


def _rigid_inverse(T):
    R = np.eye(4)
    R[:3, :3] = T[:3, :3].T
    R[:3, 3] = -T[:3, :3].T @ T[:3, 3]
    return R


def _project(T, steps):
    T = T.copy()
    for _ in range(steps):
        R = T[:3, :3]
        T[:3, :3] = 0.5 * R @ (3.0 * np.eye(3) - R.T @ R)
    return T


def _start_cost(dpt, d, P, T_init, history):
    """Cost at the start pose: too many points asked for, so nothing is updated."""
    trk = dpt.Tracker(CAM, dpt.make_params(levels=3, min_points=len(P) + 1), max_points=len(P))
    trk.set_launch_config(dpt.LAUNCH_COOP, 256)
    trk.build_pyramid(dpt.SLOT_REF, d["ref"])
    trk.set_reference_points(P, np.eye(4))
    if history is not None:
        trk.set_pose_history(*history)
    trk.build_pyramid(dpt.SLOT_CUR, d["cur"])
    trk.track_enqueue(T_init)
    r = trk.synchronize()[0]
    trk.close()
    assert r["status"] == dpt.TRACK_TOO_FEW_POINTS
    return r


@pytest.mark.parametrize("seed", range(4))
def test_prediction_from_rounded_poses(gpu_lib, seed):
    dpt = gpu_lib
    d = synth.pair(seed, cam=CAM, max_deg=0.3, max_m=0.01)
    r = np.random.default_rng(seed)
    ys, xs = r.integers(40, 440, 900), r.integers(40, 600, 900)
    P = synth.backproject(CAM, d["depth"], (ys * CAM.width + xs).astype(np.int32), np.eye(4)).astype(np.float32)
    P0 = _pose(r.uniform(-20, 20, 3), [0, 0, 0])
    P1 = np.round(_pose(0.5 * np.rad2deg(Rotation.from_matrix(P0[:3, :3]).as_rotvec()), [0, 0, 0]), 2)
    P0 = np.round(P0, 2)  # P1 P0^-1 P1 is near the identity
    start = P1 @ _rigid_inverse(P0) @ P1
    want = _start_cost(dpt, d, P, _project(start, 2), None)
    got = _start_cost(dpt, d, P, None, (P0, P1))
    assert want["n_valid_points"] > 300
    assert got["n_valid_points"] == pytest.approx(want["n_valid_points"], abs=1)
    cost = lambda q: q["final_cost"] / q["n_valid_points"]
    assert cost(got) == pytest.approx(cost(want), rel=2e-5 + 1.5 / want["n_valid_points"] * (got["n_valid_points"] != want["n_valid_points"]))
