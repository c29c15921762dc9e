"""A batch's map update (selection, back-projection, precompute) on both sides of the
rules that choose its kernels, every stream's track equal bit for bit to a plain
tracker's on the same image: the same points in the same order, the same templates.
The selection's chunks are of 1024, 4096 and 16384 candidates by the pixels of the
batch; the precompute takes one or four samples a thread and maps are dealt to XCDs
or not, by the number of maps and their size."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _same_tracks(dpt, cams, n, levels, **kw):
    import torch

    imgs, cur, depth = [], [], []
    for i, c in enumerate(cams):
        r = np.random.default_rng(100 + i)
        if i % 3 == 0:  # few grey levels: ties across chunks
            im = (r.integers(0, 3, (c.height, c.width)) * 9).astype(np.uint8)
        else:
            im = r.integers(0, 256, (c.height, c.width), dtype=np.uint8)
        imgs.append(torch.from_numpy(im).cuda())
        cur.append((imgs[-1].float() * 0.9 + 3.0).to(torch.uint8).contiguous())
        depth.append(torch.full((c.height, c.width), 2.0 + 0.01 * i, device="cuda"))
    prm = dpt.make_params(levels=levels, max_iters=2, **kw)
    eye = np.stack([np.eye(4)] * len(cams))
    bt = dpt.BatchTracker(cams, prm, [n] * len(cams))
    bt.set_launch_config(dpt.LAUNCH_COOP, 256)
    bt.build_pyramids(dpt.SLOT_REF, imgs)
    bt.set_reference_from_depth_all([n] * len(cams), depth, eye, margin=9)
    bt.build_pyramids(dpt.SLOT_CUR, cur)
    got = bt.track(eye)
    bt.close()
    for s, c in enumerate(cams):
        t = dpt.Tracker(c, prm, max_points=n)
        t.set_launch_config(dpt.LAUNCH_COOP, 256)
        t.build_pyramid(dpt.SLOT_REF, imgs[s])
        t.set_reference_from_depth(n, depth[s], np.eye(4), margin=9)
        t.build_pyramid(dpt.SLOT_CUR, cur[s])
        w = t.track(np.eye(4))
        t.close()
        assert got[s]["n_valid_points"] == w["n_valid_points"] > 0
        assert got[s]["final_cost"] == w["final_cost"]
        np.testing.assert_array_equal(np.asarray(got[s]["T_cw"]), np.asarray(w["T_cw"]))


@pytest.mark.parametrize("n_img,largest,pixels", [(5, 500, (0, 1 << 20)), (12, 900, (1 << 20, 1 << 23)),
                                                  (26, 1250, (1 << 23, 1 << 40))])
def test_selection_chunks(gpu_lib, n_img, largest, pixels):
    r = np.random.default_rng(n_img)
    cams = [synth.Camera(int(w), int(h), 400, 400, w / 2, h / 2)
            for w, h in zip(r.integers(64, largest, n_img), r.integers(64, largest, n_img))]
    cams[1] = synth.Camera(64, 66, 400, 400, 32, 33)
    cams[2] = synth.Camera(largest, largest - 1, 400, 400, largest / 2, largest / 2)
    assert pixels[0] < sum(c.width * c.height for c in cams) <= pixels[1]
    _same_tracks(gpu_lib, cams, 900, 2)


@pytest.mark.parametrize("n_img", [2, 7, 8, 9, 22])  # 22: two of 24 places idle, 9: seven of 16
@pytest.mark.parametrize("n", [500, 1100, 5000])  # 8 samples, 3 levels: 12,000 a map, 26,400 and 120,000
def test_precompute_forms(gpu_lib, n, n_img):
    cams = [synth.Camera(320 + 8 * (i % 3), 240, 250, 250, 160, 120) for i in range(n_img)]
    _same_tracks(gpu_lib, cams, n, 3)


def test_precompute_pattern_of_five(gpu_lib):
    """No multiple of four: one sample a thread at any size."""
    pat = np.array([(0, 0), (1, 2), (-2, 1), (3, -1), (-1, -3)])
    _same_tracks(gpu_lib, [synth.Camera(400, 300, 300, 300, 200, 150)] * 10, 3500, 3, pattern=pat)
