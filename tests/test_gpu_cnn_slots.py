"""The weight gradient's slots at batch sizes around their edges (one sample a
workgroup, the first layers with two, a last slot that is not full), against the
BF16-storage reference of test_gpu_cnn at its bounds, and the same batch twice:
the sums' order does not depend on timing."""
import numpy as np
import pytest

from oracle import cnn as ocnn
from test_gpu_cnn import _bf16, _bf16_storage_grads, _cos, _data, _rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def net(gpu_lib):
    p = ocnn.init_params(7)
    for i in range(1, 5):
        p[f"b{i}"] = np.random.default_rng(i).normal(0, 0.05, p[f"b{i}"].shape)
    n = gpu_lib.Cnn(max_batch=130)
    n.set_params(p)
    yield gpu_lib, n, p
    n.close()


@pytest.mark.parametrize("B", [1, 33, 64, 65, 86, 130])
def test_gradients_at_slot_edges(net, B):
    dpt, n, p = net
    pairs, tgt = _data(B, seed=B)
    loss = n.train_step(pairs, tgt, lr=0.0)
    raw = n.get_grads()
    g = dpt.cnn_unflatten(raw)
    q = {k: (_bf16(v) if k.startswith("w") else v) for k, v in p.items()}
    le, eg = _bf16_storage_grads(q, ocnn.normalise(pairs), tgt)
    assert abs(loss - le) / le < 1e-4
    for k in ocnn.PARAM_NAMES:
        assert _cos(g[k], eg[k]) > 0.99999 and _rel(g[k], eg[k]) < 2e-3, k
    assert n.train_step(pairs, tgt, lr=0.0) == loss
    np.testing.assert_array_equal(n.get_grads(), raw)
