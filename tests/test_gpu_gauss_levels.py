"""The floating-point pyramid's launches of up to three levels each, at every
split of the level count and at sizes around their tiles: equal bit for bit to
the definition in FP32 (down the columns, then across, taps in order)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _down(a):
    wt = np.array([0.125, 0.375, 0.375, 0.125], np.float32)
    h, w = a.shape
    y, x = np.arange(h // 2), np.arange(w // 2)
    col = np.zeros((h // 2, w), np.float32)
    for i in range(4):
        col = col + wt[i] * a[np.clip(2 * y - 1 + i, 0, h - 1)]
    out = np.zeros((h // 2, w // 2), np.float32)
    for j in range(4):
        out = out + wt[j] * col[:, np.clip(2 * x - 1 + j, 0, w - 1)]
    return out


@pytest.mark.parametrize("w,h,levels", [(33, 31, 1), (64, 32, 2), (65, 33, 3), (96, 95, 4), (255, 161, 5), (256, 288, 6),
                                        (545, 513, 7), (1055, 1024, 8), (1024, 1057, 8)])
def test_gauss_levels_exact(gpu_lib, w, h, levels):
    dpt = gpu_lib
    img = np.random.default_rng(w + h).integers(0, 256, (h, w), dtype=np.uint8)
    trk = dpt.Tracker(synth.Camera(w, h, 300, 300, w / 2, h / 2), dpt.make_params(levels=levels, gauss=True), max_points=8)
    trk.build_pyramid(dpt.SLOT_CUR, img)
    want, box = img.astype(np.float32), img.astype(np.int32)
    for l in range(levels):
        np.testing.assert_array_equal(trk.get_pyramid_f32(dpt.SLOT_CUR, l), want)
        np.testing.assert_array_equal(trk.get_pyramid(dpt.SLOT_CUR, l), box)
        want = _down(want)
        b = box[:box.shape[0] // 2 * 2, :box.shape[1] // 2 * 2]
        box = (b[::2, ::2] + b[1::2, ::2] + b[::2, 1::2] + b[1::2, 1::2] + 2) >> 2
    trk.close()
