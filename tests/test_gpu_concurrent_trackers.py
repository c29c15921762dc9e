"""Four trackers at once, each on its own stream with the most chunks that an
ordinary launch takes (16, all packed to one XCD) or that one with the large level
tile does (8, each with a compute unit to itself): their workgroups are resident
together on the XCD's 32 compute units, so no exchange waits for a chunk that cannot
start, and every track equals the same tracker's alone, bit for bit."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

CAM = synth.Camera(640, 480, 458.0, 458.0, 320.0, 240.0)
PATCH5 = np.stack(np.meshgrid(np.arange(-2, 3), np.arange(-2, 3)), -1).reshape(-1, 2)


@pytest.mark.parametrize("chunks", [(16, 16, 16, 16), (8, 8, 8, 8), (8, 16, 8, 16)])
@pytest.mark.parametrize("form", ["patch5", "pairs", "fp32"])
def test_four_trackers(gpu_lib, form, chunks):
    import torch

    dpt = gpu_lib
    per_chunk, kw, launch, chunk = {"patch5": (64, dict(pattern=PATCH5), dpt.LAUNCH_COOP, 256),
                                    "pairs": (128, {}, dpt.LAUNCH_COOP_PAIRS, 128),
                                    "fp32": (256, {}, dpt.LAUNCH_COOP, 256)}[form]
    tracks = 24
    trks, streams = [], [torch.cuda.Stream() for _ in range(4)]
    r = np.random.default_rng(9)
    for k, st in enumerate(streams):
        d = synth.pair(60 + k, cam=CAM, max_deg=0.4, max_m=0.01)
        points = per_chunk * chunks[k]
        ys, xs = r.integers(16, 464, points), r.integers(16, 624, points)
        P = synth.backproject(CAM, d["depth"], (ys * CAM.width + xs).astype(np.int32), np.eye(4)).astype(np.float32)
        trk = dpt.Tracker(CAM, dpt.make_params(levels=3, **kw), max_points=points, stream=st.cuda_stream)
        trk.set_launch_config(launch, chunk)
        trk.build_pyramid(dpt.SLOT_REF, d["ref"])
        trk.set_reference_points(P, np.eye(4))
        trk.build_pyramid(dpt.SLOT_CUR, d["cur"])
        trks.append(trk)
    alone = [t.track(np.eye(4)) for t in trks]
    for _ in range(tracks):
        for t in trks:
            t.track_enqueue(np.eye(4))
    for t, want in zip(trks, alone):
        got = t.synchronize()
        assert len(got) == tracks
        for g in got:
            assert g["status"] == want["status"] != dpt.TRACK_TIMEOUT
            np.testing.assert_array_equal(np.asarray(g["T_cw"]), np.asarray(want["T_cw"]))
            assert g["final_cost"] == want["final_cost"] and g["iterations"] == want["iterations"]
        t.close()
