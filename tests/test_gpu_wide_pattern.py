"""Eight samples that reach 16 pixels each way on frames wide enough that the
pattern's rows are more than a workgroup's level tile holds: points that turn
unusable (and those that are from the start) read nothing past the tile, and the
track meets the FP64 oracle's bar."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

PATTERN = np.array([(0, 0), (-16, -16), (16, 16), (16, -16), (-16, 16), (0, 16), (0, -16), (5, 2)], np.int32)


@pytest.mark.parametrize("form", ["fp32", "pairs", "mixed", "fixed_h"])
@pytest.mark.parametrize("width", [1820, 1860, 2048])  # below, just past and beyond the tile at level 0
def test_pattern_past_the_tile(gpu_lib, width, form):
    dpt = gpu_lib
    cam = synth.Camera(width, 200, 0.7 * width, 0.7 * width, width / 2, 100.0)
    d = synth.pair(31, cam=cam, max_deg=0.3, max_m=0.01)
    n = 600
    r = np.random.default_rng(width)
    ys, xs = r.integers(18, 182, n), r.integers(18, width - 18, n)
    P = synth.backproject(cam, d["depth"], (ys * width + xs).astype(np.int32), np.eye(4)).astype(np.float32)
    P[100:300, 2] *= -1.0  # whole waves behind the camera
    kw = dict(fixed_h=True) if form == "fixed_h" else dict(precision=dpt.PREC_MIXED) if form == "mixed" else {}
    trk = dpt.Tracker(cam, dpt.make_params(levels=3, pattern=PATTERN, **kw), max_points=n)
    trk.set_launch_config(dpt.LAUNCH_COOP_PAIRS if form == "pairs" else dpt.LAUNCH_COOP, 64)
    trk.build_pyramid(dpt.SLOT_REF, d["ref"])
    trk.set_reference_points(P, np.eye(4))
    trk.build_pyramid(dpt.SLOT_CUR, d["cur"])
    g = trk.track(np.eye(4))
    trk.close()
    prm = oracle.make_params(levels=3, pattern=PATTERN, **(dict(fixed_h=True) if form == "fixed_h" else {}))
    o = oracle.Reference(cam, prm, d["ref"], P, np.eye(4)).track(d["cur"], np.eye(4))
    rot, tr = oracle.pose_error(g["T_cw"], o["T_cw"])
    assert g["status"] == o["status"]
    assert rot < 1e-4 and tr < 1e-4, (rot, tr)
    assert abs(g["final_cost"] - o["final_cost"]) <= 1e-3 * max(o["final_cost"], 1e-3)
    assert g["n_valid_points"] == pytest.approx(o["n_valid_points"], abs=1)
