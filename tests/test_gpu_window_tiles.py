"""Window pyramids by one, two and four tiles of a row per workgroup (3072 tiles in a
launch and fewer, or more with rows of 5 and of 11 tiles): every frame's track equal
bit for bit to that of a plain tracker that builds the frame's pyramid by itself."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


# 315 x 251: rows of 5 tiles; 641 x 479: of 11, both odd so that no row starts aligned
@pytest.mark.parametrize("w,h,streams,frames", [(315, 251, 3, 4), (315, 251, 20, 9), (641, 479, 2, 4), (641, 479, 6, 7)])
def test_window_pyramids(gpu_lib, w, h, streams, frames):
    import torch

    dpt = gpu_lib
    cam = synth.Camera(w, h, 300.0, 300.0, w / 2, h / 2)
    d = synth.pair(6, cam, max_deg=0.3, max_m=0.01)
    n = 200
    P = synth.backproject(cam, d["depth"], oracle.select_points(d["ref"], n, 8), d["T_rw"])
    r = np.random.default_rng(0)
    # every frame other noise, so that a tile of a wrong frame shows
    stack = np.clip(d["cur"][None, None] + r.integers(-3, 4, (streams, frames, h, w)), 0, 255).astype(np.uint8)
    dev = torch.from_numpy(stack).cuda()
    prm = dpt.make_params(levels=5)
    start = np.stack([np.eye(4)] * streams)
    bt = dpt.BatchTracker([cam] * streams, prm, [n] * streams)
    bt.set_launch_config(dpt.LAUNCH_COOP, 256)
    bt.build_pyramids(dpt.SLOT_REF, [torch.from_numpy(d["ref"]).cuda()] * streams)
    for s in range(streams):
        bt.set_reference_points(s, P, d["T_rw"])
    bt.set_pose_history_all(start, start)
    bt.track_window_enqueue(dev)
    got = bt.collect(frames)
    bt.close()
    for s in sorted({0, 1, streams - 1}):
        t = dpt.Tracker(cam, prm, max_points=n)
        t.set_launch_config(dpt.LAUNCH_COOP, 256)
        t.build_pyramid(dpt.SLOT_REF, d["ref"])
        t.set_reference_points(P, d["T_rw"])
        t.set_pose_history(np.eye(4), np.eye(4))
        for f in range(frames):
            t.build_pyramid(dpt.SLOT_CUR, dev[s, f])
            t.track_enqueue()
            w1 = t.collect(1)[0]
            np.testing.assert_array_equal(np.asarray(got[f][s]["T_cw"]), np.asarray(w1["T_cw"]))
            assert got[f][s]["final_cost"] == w1["final_cost"]
        t.close()
