"""The cooperative track's exchange and lane-parallel solve at the edges of their
ranges: chunk counts around the lane groups (2 of 32 values, 4 of 16 in the
fixed-H mode) and the poll batches of 8 chunks each, maps that fill the last
chunk or leave it almost empty, and a start so far off that the first updates
take the large-angle branch of the exponential (more than 0.05 rad).  Against
the FP64 oracle, at the tracker's bar."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

CAM = synth.Camera(320, 240, 230.0, 230.0, 160.0, 120.0)


@pytest.fixture(scope="module")
def pair():
    return synth.pair(4242, cam=CAM, max_deg=0.6, max_m=0.015)


def _track(dpt, d, n, T_init, chunk, **kw):
    trk = dpt.Tracker(CAM, dpt.make_params(levels=3, **kw), max_points=n)
    trk.set_launch_config(dpt.LAUNCH_COOP, chunk)
    trk.build_pyramid(dpt.SLOT_REF, d["ref"])
    idx = trk.select_points(n, 8)
    P = synth.backproject(CAM, d["depth"], idx, d["T_rw"])
    trk.set_reference_points(P, d["T_rw"])
    trk.build_pyramid(dpt.SLOT_CUR, d["cur"])
    r = trk.track(T_init)
    trk.close()
    return r, P


def _assert_close(r, o):
    E = np.asarray(r["T_cw"]) @ np.linalg.inv(o["T_cw"])
    s = 0.5 * np.linalg.norm([E[2, 1] - E[1, 2], E[0, 2] - E[2, 0], E[1, 0] - E[0, 1]])
    assert r["status"] == o["status"]
    assert s < 1e-4 and np.linalg.norm(E[:3, 3]) < 1e-4, (s, E[:3, 3])
    assert abs(r["final_cost"] - o["final_cost"]) <= 1e-3 * max(o["final_cost"], 1e-3)
    assert r["n_valid_points"] == pytest.approx(o["n_valid_points"], abs=1)


@pytest.mark.parametrize("mode", ["fp32", "mixed", "fixed_h"])
@pytest.mark.parametrize("n", [60, 64, 65, 190, 512, 513, 1024, 1025, 2100])  # 1, 1, 2, 3, 8, 9, 16, 17, 33 chunks
def test_chunk_counts(gpu_lib, pair, n, mode):
    dpt = gpu_lib
    kw = dict(precision=dpt.PREC_MIXED) if mode == "mixed" else dict(fixed_h=mode == "fixed_h")
    r, P = _track(dpt, pair, n, np.eye(4), 64, **kw)
    prm = oracle.make_params(levels=3, **({"fixed_h": True} if mode == "fixed_h" else {}))
    o = oracle.Reference(CAM, prm, pair["ref"], P, pair["T_rw"]).track(pair["cur"], np.eye(4))
    _assert_close(r, o)


@pytest.mark.parametrize("mode", ["fp32", "mixed", "fixed_h"])
def test_large_angle_update(gpu_lib, pair, mode):
    """A roll of 4 degrees about the optical axis: the first coarse update turns by about as much."""
    from scipy.spatial.transform import Rotation

    dpt = gpu_lib
    T0 = synth.pose_matrix(Rotation.from_rotvec([0.0, 0.0, np.deg2rad(4.0)]).as_matrix(), np.zeros(3))
    kw = dict(precision=dpt.PREC_MIXED) if mode == "mixed" else dict(fixed_h=mode == "fixed_h")
    r, P = _track(dpt, pair, 1500, T0, 256, **kw)
    prm = oracle.make_params(levels=3, **({"fixed_h": True} if mode == "fixed_h" else {}))
    o = oracle.Reference(CAM, prm, pair["ref"], P, pair["T_rw"]).track(pair["cur"], T0)
    _assert_close(r, o)
