"""The precompute with four samples to a thread and the maps of a batch dealt to
XCDs: every template of the large map equal bit for bit to the same points in a
small map (one sample to a thread), and batches whose size is no multiple of
eight equal to plain trackers."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def _cache(dpt, cam, img, P, T, levels, **kw):
    t = dpt.Tracker(cam, dpt.make_params(levels=levels, **kw), max_points=len(P))
    t.build_pyramid(dpt.SLOT_REF, img)
    t.set_reference_points(P, T)
    out = [t.reference_cache(l) for l in range(levels)]
    t.close()
    return out


@pytest.mark.parametrize("kw", [{}, dict(precision=1), dict(pattern=np.array([(0, 0), (1, -2), (-3, 1), (2, 2)])),
                                dict(gauss=True, pattern=np.array([(i % 4 - 1, i // 4 - 1) for i in range(12)]))])
def test_four_samples_equal_one(gpu_lib, kw):
    dpt = gpu_lib
    cam, levels = synth.CAM_1280, 6
    d = synth.pair(31, cam)
    n = 16000
    P = synth.backproject(cam, d["depth"], oracle.select_points(d["ref"], n, 8), d["T_rw"])
    P[5], P[-1] = np.nan, (0, 0, -1e3)  # no reference: zero templates on either path
    big = _cache(dpt, cam, d["ref"], P, d["T_rw"], levels, **kw)
    for lo in (0, 7999, n - 500):  # small maps: well below the rule's 2^18 samples over all levels
        part = _cache(dpt, cam, d["ref"], P[lo:lo + 500], d["T_rw"], levels, **kw)
        for b, s in zip(big, part):
            for k in s:
                np.testing.assert_array_equal(np.asarray(b[k])[lo:lo + 500], s[k], err_msg=k)


@pytest.mark.parametrize("n_img", [1, 7, 9, 17])
def test_batches_of_any_size(gpu_lib, n_img):
    import torch

    dpt = gpu_lib
    cam, n = synth.CAM_640, 300 if n_img < 17 else 4000  # one sample a thread, four
    d = synth.pair(32, cam)
    ref, cur = torch.from_numpy(d["ref"]).cuda(), torch.from_numpy(d["cur"]).cuda()
    depth = torch.from_numpy(np.asarray(d["depth"], np.float32)).cuda()
    prm = dpt.make_params(levels=3)
    bt = dpt.BatchTracker([cam] * n_img, prm, [n] * n_img)
    bt.build_pyramids(dpt.SLOT_REF, [ref] * n_img)
    bt.set_reference_from_depth_all([n] * n_img, [depth] * n_img, np.stack([d["T_rw"]] * n_img))
    bt.build_pyramids(dpt.SLOT_CUR, [cur] * n_img)
    got = bt.track(np.stack([np.eye(4)] * n_img))
    bt.close()
    t = dpt.Tracker(cam, prm, max_points=n)
    t.build_pyramid(dpt.SLOT_REF, ref)
    t.set_reference_from_depth(n, depth, d["T_rw"])
    t.build_pyramid(dpt.SLOT_CUR, cur)
    w = t.track(np.eye(4))
    t.close()
    for g in got:
        rot, tr = oracle.pose_error(g["T_cw"], w["T_cw"])
        assert rot < 1e-5 and tr < 1e-5 and g["n_valid_points"] == w["n_valid_points"]
