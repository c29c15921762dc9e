"""Patterns whose templates the cooperative track keeps in registers, at the
edges of that form: sample counts around the lane slots (7 x 4, 13 x 4) and past
them, on the uint8 and the floating-point pyramid, and offsets that span more
rows of a wide floating-point level than the workgroup's LDS tile holds.
Against the FP64 oracle, at the tracker's bar."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def _pattern(k, reach=5):
    """k distinct offsets within `reach`, the centre and two far corners first."""
    r = np.arange(-reach, reach + 1)
    g = np.stack(np.meshgrid(r, r), -1).reshape(-1, 2)
    g = g[np.random.default_rng(reach).permutation(len(g))]
    first = np.array([(0, 0), (-reach, -reach), (reach, reach)])
    rest = g[~(g[:, None] == first[None]).all(-1).any(1)]
    return np.concatenate([first, rest])[:k].astype(np.int32)


def _check(dpt, cam, n, seed, pat, gauss, fixed_h):
    d = synth.pair(seed, cam)
    idx = oracle.select_points(d["ref"], n, 20)
    P = synth.backproject(cam, d["depth"], idx, d["T_rw"])
    trk = dpt.Tracker(cam, dpt.make_params(levels=3, pattern=pat, gauss=gauss, fixed_h=fixed_h), max_points=n)
    trk.set_launch_config(dpt.LAUNCH_COOP, 256)
    trk.build_pyramid(dpt.SLOT_REF, d["ref"])
    trk.set_reference_points(P, d["T_rw"])
    trk.build_pyramid(dpt.SLOT_CUR, d["cur"])
    g = trk.track(np.eye(4))
    trk.close()
    prm = oracle.make_params(levels=3, pattern=pat, gauss=gauss, fixed_h=fixed_h)
    o = oracle.Reference(cam, prm, d["ref"], P, d["T_rw"]).track(d["cur"], np.eye(4))
    rot, tr = oracle.pose_error(g["T_cw"], o["T_cw"])
    assert g["status"] == o["status"]
    assert rot < 1e-4 and tr < 1e-4, (rot, tr)
    assert abs(g["final_cost"] - o["final_cost"]) <= 1e-3 * max(o["final_cost"], 1e-3)
    assert g["n_valid_points"] == pytest.approx(o["n_valid_points"], abs=1)


@pytest.mark.parametrize("gauss", [False, True])
@pytest.mark.parametrize("fixed_h", [False, True])
@pytest.mark.parametrize("k", [3, 4, 27, 28, 29, 51, 52, 53, 56])
def test_pattern_sizes(gpu_lib, k, fixed_h, gauss):
    _check(gpu_lib, synth.CAM_640, 330, 12, _pattern(k), gauss, fixed_h)


@pytest.mark.parametrize("fixed_h", [False, True])
def test_rows_past_the_tile(gpu_lib, fixed_h):
    _check(gpu_lib, synth.CAM_1280, 700, 15, _pattern(40, 16), True, fixed_h)
