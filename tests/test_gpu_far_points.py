"""A map point that no level holds as valid adds nothing to its stream, wherever
it lies: points so far to the side that their Jacobian rows overflow FP32 (or
so near that 1/z does) give the same tracks, bit for bit, as points behind the
camera in their places.  Every form of the cooperative kernel, over two frames
(the second starts from the first's pose)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

CAM = synth.Camera(320, 240, 230.0, 230.0, 160.0, 120.0)
BIG = np.float32(3e38)
FAR = np.array([(1e30, 1e30, 5.0), (-1e30, 3.0, 5.0), (2.0, 4e19, 1.0), (BIG, -BIG, 0.5)], np.float32)
NEAR = np.array([(0.0, 0.0, 1e-40), (1.0, 0.0, 1e-30), (1e-3, 1e-3, 1e-42)], np.float32)
FORMS = {
    "fp32": ({}, "coop"),
    "mixed": (dict(precision=1), "coop"),
    "fixed_h": (dict(fixed_h=True), "coop"),
    "pairs": ({}, "pairs"),
    "pairs_mixed": (dict(precision=1), "pairs"),
    "pairs_fixed_h": (dict(fixed_h=True), "pairs"),
    "patch5": (dict(patch=5), "coop"),
    "patch5_fixed_h": (dict(patch=5, fixed_h=True), "coop"),
    "patch9": (dict(patch=9), "coop"),
    "gauss": (dict(gauss=True), "coop"),
}


@pytest.fixture(scope="module")
def pair():
    return synth.pair(77, cam=CAM, max_deg=0.5, max_m=0.01)


def _tracks(dpt, d, kw, launch, P):
    kw = dict(kw)
    side = kw.pop("patch", 0)
    if side:
        r = np.arange(side) - side // 2
        kw["pattern"] = np.stack(np.meshgrid(r, r), -1).reshape(-1, 2)
    trk = dpt.Tracker(CAM, dpt.make_params(levels=3, **kw), max_points=len(P))
    trk.set_launch_config(dpt.LAUNCH_COOP if launch == "coop" else dpt.LAUNCH_COOP_PAIRS, 128)
    trk.build_pyramid(dpt.SLOT_REF, d["ref"])
    trk.set_reference_points(P, d["T_rw"])
    trk.build_pyramid(dpt.SLOT_CUR, d["cur"])
    trk.set_pose_history(np.eye(4), np.eye(4))
    out = []
    for _ in range(2):  # the second from the history that the first extended
        trk.track_enqueue(None)
        out.append(trk.synchronize()[0])
    trk.close()
    return out


@pytest.mark.parametrize("z_min", [1e-3, 0.0])
@pytest.mark.parametrize("form", sorted(FORMS))
def test_far_points_are_left_out(gpu_lib, pair, form, z_min):
    dpt = gpu_lib
    kw, launch = FORMS[form]
    kw = dict(kw, z_min=z_min)
    n = 700
    # map points of the scene, in no order, and odd ones among them
    r = np.random.default_rng(5)
    ys, xs = r.integers(12, 228, n), r.integers(12, 308, n)
    P = synth.backproject(CAM, pair["depth"], (ys * CAM.width + xs).astype(np.int32), np.eye(4)).astype(np.float32)
    odd = np.concatenate([FAR, NEAR]) if z_min == 0.0 else FAR
    at = 3 + 83 * np.arange(len(odd))
    behind, far = P.copy(), P.copy()
    behind[at] = (0.1, 0.1, -1.0)
    far[at] = odd
    d = dict(pair, T_rw=np.eye(4))
    want = _tracks(dpt, d, kw, launch, behind)
    got = _tracks(dpt, d, kw, launch, far)
    for a, b in zip(got, want):
        assert b["status"] in (dpt.TRACK_OK, dpt.TRACK_MAX_ITERS)
        assert a["status"] == b["status"] and a["iterations"] == b["iterations"]
        assert a["n_valid_points"] == b["n_valid_points"]
        np.testing.assert_array_equal(np.asarray(a["T_cw"]), np.asarray(b["T_cw"]))
        assert a["final_cost"] == b["final_cost"]
