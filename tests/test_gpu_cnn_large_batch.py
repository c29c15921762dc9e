"""The sums over a training batch far above 256: a batch of B copies of one pair (B
a power of two, so every scaled value is the single pair's exactly) has the single
pair's gradient, but for the rounding of its sums.  Bound per tensor, on the rms:
B / 64 values in one chain up to 1024 copies and B / 256 above, of equal sign and
size, round off at most 2^-25 of the sum each."""
import numpy as np
import pytest

from oracle import cnn as ocnn
from test_gpu_cnn import _bf16, _bf16_storage_grads, _cos, _data, _rel

pytestmark = pytest.mark.gpu

SHAPES = [("w1", 16 * 18), ("b1", 16), ("w2", 32 * 144), ("b2", 32), ("w3", 64 * 288), ("b3", 64), ("w4", 64 * 576),
          ("b4", 64), ("fw1", 4096), ("fb1", 64), ("fw2", 384), ("fb2", 6)]

def _errors(dpt, B):
    """rms error of each tensor's gradient of B copies, relative to its rms."""
    import torch

    assert sum(n for _, n in SHAPES) == dpt.load().dpt_cnn_num_params()
    r = np.random.default_rng(B)
    w = np.concatenate([r.normal(0, 0.05 if k.startswith("b") or k.startswith("fb") else np.sqrt(2.0 / max(n // 64, 9)), n)
                        for k, n in SHAPES]).astype(np.float32)
    shade = r.normal(128, 40, (1, 1, 60, 94))
    pair = np.clip(shade + r.normal(0, 12, (1, 2, 60, 94)), 0, 255).astype(np.uint8)
    target = r.normal(0, 0.3, (1, 6)).astype(np.float32)
    grads = []
    for n in (1, B):
        net = dpt.Cnn(max_batch=n)
        net.set_params(w)
        net.train_step(torch.from_numpy(pair).cuda().repeat(n, 1, 1, 1), torch.from_numpy(target).cuda().repeat(n, 1), 0.0)
        grads.append(net.get_grads().astype(np.float64))
        net.close()
    out, at = {}, 0
    for k, n in SHAPES:
        one, many = grads[0][at:at + n], grads[1][at:at + n]
        assert np.sqrt(np.mean(one ** 2)) > 0, k
        out[k] = np.sqrt(np.mean((many - one) ** 2) / np.mean(one ** 2))
        at += n
    return out

def _bound(B):
    return 2.0 ** -25 * (B / 64 if B <= 1024 else B / 256)

@pytest.mark.parametrize("B", [1024, 4096, 16384])
def test_fc_gradients(gpu_lib, B):
    e = _errors(gpu_lib, B)
    bad = {k: e[k] for k in ("fw1", "fb1", "fw2", "fb2") if not e[k] <= _bound(B)}
    assert not bad, (bad, _bound(B))


@pytest.mark.parametrize("B", [512, 1024, 4096, 16384])
def test_conv_gradients(gpu_lib, B):
    e = _errors(gpu_lib, B)
    bad = {k: v for k, v in e.items() if k not in ("fw1", "fb1", "fw2", "fb2") and not v <= _bound(B)}
    assert not bad, (bad, _bound(B))


def test_ragged_last_workgroup(gpu_lib):
    """513 pairs: one sample, or three, in the last workgroup of each layer; against
    the BF16-storage reference of test_gpu_cnn at its bounds."""
    p = ocnn.init_params(7)
    pairs, tgt = _data(513, seed=513)
    net = gpu_lib.Cnn(max_batch=513)
    net.set_params(p)
    loss = net.train_step(pairs, tgt, lr=0.0)
    g = gpu_lib.cnn_unflatten(net.get_grads())
    net.close()
    le, eg = _bf16_storage_grads({k: (_bf16(v) if k.startswith("w") else v) for k, v in p.items()},
                                 ocnn.normalise(pairs), tgt)
    assert abs(loss - le) / le < 1e-4
    for k in ocnn.PARAM_NAMES:
        assert _cos(g[k], eg[k]) > 0.99999 and _rel(g[k], eg[k]) < 2e-3, k
