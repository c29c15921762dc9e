"""The level tile's size follows how the map was set: a selected map (index order)
takes the small tile unless its chunks span more than the large one, points given by
the caller the large one up to eight chunks.  The same points set either way give the
same track, bit for bit, frame and window forms."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

FORMS = {"fp32": ({}, "coop"), "mixed": (dict(precision=1), "coop"), "fixed_h": (dict(fixed_h=True), "coop"),
         "pairs": ({}, "pairs"), "patch5": (dict(patch=5), "coop"), "gauss7": (dict(patch=7, gauss=True), "coop")}


@pytest.mark.parametrize("w,h,n", [(320, 240, 300), (752, 480, 200), (752, 480, 1000), (1280, 720, 150), (1280, 720, 500)])
@pytest.mark.parametrize("form", sorted(FORMS))
def test_selected_equals_given(gpu_lib, form, w, h, n):
    import torch

    dpt = gpu_lib
    kw, launch = FORMS[form]
    kw = dict(kw)
    side = kw.pop("patch", 0)
    if side:
        r = np.arange(side) - side // 2
        kw["pattern"] = np.stack(np.meshgrid(r, r), -1).reshape(-1, 2)
        n = min(n, 500)  # chunks of 64 points: eight at most
    cam = synth.Camera(w, h, 0.62 * w, 0.62 * w, w / 2, h / 2)
    d = synth.pair(9, cam=cam, max_deg=0.4, max_m=0.015)
    frames = torch.from_numpy(np.stack([d["cur"], d["ref"], d["cur"]])).cuda()
    depth = np.asarray(d["depth"], np.float32)
    out, x0 = [], None
    for given in (False, True):
        t = dpt.Tracker(cam, dpt.make_params(levels=4, **kw), max_points=n)
        t.set_launch_config(dpt.LAUNCH_COOP_PAIRS if launch == "pairs" else dpt.LAUNCH_COOP, 128 if launch == "pairs" else 256)
        t.build_pyramid(dpt.SLOT_REF, d["ref"])
        if given:
            t.set_reference_points(x0, np.eye(4))
        else:
            t.set_reference_from_depth(n, depth, np.eye(4), margin=10)
            x0 = t.reference_cache(0)["x0"].copy()  # at the identity: the map itself
        t.build_pyramid(dpt.SLOT_CUR, d["cur"])
        res = [t.track(np.eye(4))]
        if "gauss" not in form:
            t.set_pose_history(np.eye(4), np.eye(4))
            t.track_window_enqueue(frames)
            res += t.collect(3)
        out.append(res)
        t.close()
    assert out[0][0]["n_valid_points"] > n // 2
    for a, b in zip(*out):
        assert a["status"] == b["status"] and a["iterations"] == b["iterations"]
        np.testing.assert_array_equal(np.asarray(a["T_cw"]), np.asarray(b["T_cw"]))
        assert a["final_cost"] == b["final_cost"]
