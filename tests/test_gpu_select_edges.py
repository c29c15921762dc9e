"""Selection at the edges of its groups, chunks and launches: rows whose length
is no multiple of four (a group spans two rows), odd pitches and first bytes,
images on either side of the chunk sizes' limit, a flat image (every candidate
ties), one of few grey levels (ties across chunks), and more wanted than there
are candidates.  Equal to the definition, twice in a row on the same scratch."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def _image(kind, h, w, seed):
    r = np.random.default_rng(seed)
    if kind == "flat":
        return np.full((h, w), 77, np.uint8)
    if kind == "few":
        return (r.integers(0, 3, (h, w)) * 9).astype(np.uint8)
    return r.integers(0, 256, (h, w), dtype=np.uint8)


@pytest.mark.parametrize("kind", ["noise", "few", "flat"])
@pytest.mark.parametrize("w,h,margin,pad", [(3, 3, 1, 0), (5, 4, 1, 2), (67, 41, 3, 1), (130, 70, 8, 3), (641, 479, 5, 2),
                                            (1024, 1024, 4, 0), (1025, 1024, 1, 4), (1031, 1200, 6, 1), (2900, 2903, 2, 1)])
def test_select_edges(gpu_lib, w, h, margin, pad, kind):
    import torch

    dpt = gpu_lib
    cand = (w - 2 * margin) * (h - 2 * margin)
    img = _image(kind, h, w, w + h)
    buf = torch.zeros(h * (w + pad) + 1, dtype=torch.uint8, device="cuda")
    view = buf[1:].view(h, w + pad)[:, :w]  # rows from an odd address
    view.copy_(torch.from_numpy(img))
    for n in sorted({1, min(cand, 1000), cand, min(w * h, cand + 5)}):
        want = oracle.select_points(img, n, margin)
        for _ in range(2):
            idx = torch.full((n,), -1, dtype=torch.int32, device="cuda")
            cnt = torch.zeros(1, dtype=torch.int32, device="cuda")
            dpt.select_points_noalloc(view, n, margin, idx, cnt)
            torch.cuda.synchronize()
            got = idx.cpu().numpy()
            assert int(cnt) == len(want)
            np.testing.assert_array_equal(got[:len(want)], want)
            assert (got[len(want):] == -1).all()


@pytest.mark.parametrize("n_img", [2, 5, 40])  # small chunks, large ones, the histograms' least workgroups per image
def test_batch_selection_equals_plain(gpu_lib, n_img):
    """The maps of a batch's keyframes, seen through one Gauss-Newton step on
    each: the same points give the same valid counts, and costs and poses that
    differ by FP32 summation order only."""
    import torch

    dpt = gpu_lib
    r = np.random.default_rng(n_img)
    cams = [synth.Camera(int(w), int(h), 400, 400, w / 2, h / 2)
            for w, h in zip(r.integers(64, 700, n_img), r.integers(64, 500, n_img))]
    imgs = [torch.from_numpy(_image("few" if i % 3 == 0 else "noise", c.height, c.width, i)).cuda()
            for i, c in enumerate(cams)]
    cur = [(im.float() * 0.9 + 3.0).to(torch.uint8).contiguous() for im in imgs]
    depth = [torch.full((c.height, c.width), 2.0, device="cuda") for c in cams]
    prm = dpt.make_params(levels=2, max_iters=1)
    n, eye = 700, np.stack([np.eye(4)] * n_img)
    bt = dpt.BatchTracker(cams, prm, [n] * n_img)
    bt.build_pyramids(dpt.SLOT_REF, imgs)
    bt.set_reference_from_depth_all([n] * n_img, depth, eye, margin=9)
    bt.build_pyramids(dpt.SLOT_CUR, cur)
    got = bt.track(eye)
    bt.close()
    for s, c in enumerate(cams):
        t = dpt.Tracker(c, prm, max_points=n)
        t.build_pyramid(dpt.SLOT_REF, imgs[s])
        t.set_reference_from_depth(n, depth[s], np.eye(4), margin=9)
        t.build_pyramid(dpt.SLOT_CUR, cur[s])
        w = t.track(np.eye(4))
        t.close()
        assert got[s]["n_valid_points"] == w["n_valid_points"]
        assert got[s]["final_cost"] == pytest.approx(w["final_cost"], rel=1e-4)
        rot, tr = oracle.pose_error(got[s]["T_cw"], w["T_cw"])
        assert rot < 1e-5 and tr < 1e-5
