"""The 64x64-tile pyramid at any width, pitch and first byte: widths around its
16-byte pieces and its tiles, rows from odd addresses, in a plain, a batched and a
window build; equal byte for byte to the definition."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def _view(img, pad, lead):
    """The device bytes from img's first pixel on, rows w + pad apart, the first at byte `lead` of its allocation."""
    import torch

    h, w = img.shape
    buf = torch.zeros(lead + h * (w + pad), dtype=torch.uint8, device="cuda")
    buf[lead:].view(h, w + pad)[:, :w].copy_(torch.from_numpy(img))
    return buf[lead:]


@pytest.mark.parametrize("pad,lead", [(0, 0), (3, 1), (1, 7)])
@pytest.mark.parametrize("w,h,levels", [(16, 19, 1), (17, 16, 2), (31, 33, 2), (63, 65, 3), (64, 64, 4), (65, 63, 3), (79, 66, 4),
                                        (131, 128, 5), (641, 479, 4), (530, 1030, 7)])
def test_plain_and_batch(gpu_lib, w, h, levels, pad, lead):
    dpt = gpu_lib
    cam = synth.Camera(w, h, 200, 200, w / 2, h / 2)
    imgs = [np.random.default_rng(w + i).integers(0, 256, (h, w), dtype=np.uint8) for i in range(3)]
    prm = dpt.make_params(levels=levels)
    t = dpt.Tracker(cam, prm, max_points=8)
    v = _view(imgs[0], pad, lead)
    t.build_pyramid(dpt.SLOT_CUR, v, pitch=w + pad)
    for l, want in enumerate(oracle.pyramid(imgs[0], levels)):
        np.testing.assert_array_equal(t.get_pyramid(dpt.SLOT_CUR, l), want)
    t.close()
    bt = dpt.BatchTracker([cam] * 3, prm, [8] * 3)
    bt.build_pyramids(dpt.SLOT_CUR, [_view(i, pad, lead) for i in imgs], pitches=[w + pad] * 3)
    for l in range(levels):
        got = bt.get_level(dpt.SLOT_CUR, l)
        got = got.cpu().numpy() if hasattr(got, "cpu") else np.asarray(got)
        for k, i in enumerate(imgs):
            np.testing.assert_array_equal(got[k].reshape(-1)[:(w >> l) * (h >> l)].reshape(h >> l, w >> l),
                                          oracle.pyramid(i, levels)[l])
    bt.close()


@pytest.mark.parametrize("w,h", [(641, 479), (333, 251)])
def test_window_equals_frames(gpu_lib, w, h):
    import torch

    dpt = gpu_lib
    cam = synth.Camera(w, h, 300.0, 300.0, w / 2, h / 2)
    d = synth.pair(5, cam, max_deg=0.3, max_m=0.01)
    idx = oracle.select_points(d["ref"], 500, 8)
    P = synth.backproject(cam, d["depth"], idx, d["T_rw"])
    frames = [d["cur"], d["ref"], d["cur"]]
    stack = torch.from_numpy(np.stack(frames)).cuda()
    res = []
    for windowed in (True, False):
        t = dpt.Tracker(cam, dpt.make_params(levels=3), max_points=500)
        t.build_pyramid(dpt.SLOT_REF, d["ref"])
        t.set_reference_points(P, d["T_rw"])
        t.set_pose_history(np.eye(4), np.eye(4))
        if windowed:
            t.track_window_enqueue(stack)
            res.append(t.collect(3))
        else:
            out = []
            for k in range(3):
                t.build_pyramid(dpt.SLOT_CUR, stack[k])
                t.track_enqueue()
                out += t.collect(1)
            res.append(out)
        t.close()
    for a, b in zip(*res):
        np.testing.assert_array_equal(np.asarray(a["T_cw"]), np.asarray(b["T_cw"]))
        assert a["final_cost"] == b["final_cost"] and a["status"] == b["status"]
