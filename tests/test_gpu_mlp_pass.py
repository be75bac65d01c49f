"""The network's fused passes at the sizes where their split changes: ragged last row blocks, one to eight shares of
the outputs, and the batch in one or two halves for the weight gradients.  References and tolerances as in
test_gpu_mlp.py: the oracle's network with the same bfloat16 rounding points, where an FP32 sum close to a rounding
boundary moves single rows by 1e-3 and whole batches by less than 5e-4 (outputs) and 1e-3 (gradients)."""
import numpy as np
import pytest

from oracle import surrogate as S
from synth import generators as gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1307_3424_amd as wp  # noqa: E402


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def feat(n):
    return np.random.default_rng(n).uniform(-1, 1, (n, 3)).astype(np.float32)


# 2017 and 4100 rows: 64 and 129 blocks of 32, eight and four shares; 8200: two shares; 16384: one
@pytest.mark.parametrize("n", [31, 33, 2017, 4100, 8200, 16384])
def test_forward_of_ragged_batches(n):
    m = wp.Mlp(max_batch=(n + 63) // 64 * 64)
    p = gen.mlp_init(21)
    m.set_params(p, 1.0, 1.0)
    X = feat(n)
    out = m.forward(dev(X.ravel())).cpu().numpy().reshape(n, -1)
    m.close()
    rows = np.unique(np.concatenate([np.arange(min(n, 40)), np.arange(max(0, n - 40), n)]))
    ref, _ = S.forward(S.from_packed(p), X[rows].astype(np.float64), q=S.round_bf16)
    assert np.linalg.norm(out[rows] - ref) / np.linalg.norm(ref) < 5e-4
    assert (np.linalg.norm(out[rows] - ref, axis=1) / np.linalg.norm(ref, axis=1)).max() < 3e-3


@pytest.mark.parametrize("n", [64, 1984, 2048, 2112])
def test_gradients_in_one_and_two_halves(n):
    m = wp.Mlp(max_batch=2112)
    p = gen.mlp_init(22)
    m.set_params(p, 1.0, 1.0)
    X = feat(n)
    T = np.random.default_rng(n + 1).normal(size=(n, 2048)).astype(np.float32) * 0.05
    for _ in range(2):                                        # the second call starts from the first one's gradients
        g, loss = m.gradients(dev(X.ravel()), dev(T.ravel()))
    g = g.cpu().numpy()
    m.close()
    net = S.from_packed(p)
    o, cache = S.forward(net, X.astype(np.float64), q=S.round_bf16)
    l_ref, dO = S.mse_loss(o, T.astype(np.float64))
    ref = S.backward(net, cache, dO, q=S.round_bf16)
    assert abs(loss - l_ref) <= 1e-5 * l_ref
    for k in net.NAMES:
        a, b = getattr(S.from_packed(g), k), ref[k]
        assert np.linalg.norm(a - b) <= 1e-3 * np.linalg.norm(b), k


def test_gelu_of_large_and_small_arguments():
    """One hidden unit's path, far outside the trained range: gelu(x) = x for large x, 0 for very negative x."""
    net = S.from_packed(np.zeros(wp.Mlp.param_count(), dtype=np.float32))
    net.W1[0, 0] = 1.0
    net.W2[0, 0] = net.W3[0, 0] = 1.0
    net.W4[0, 0] = 1.0
    p = np.concatenate([getattr(net, k).ravel() for k in ("W1", "b1", "W2", "b2", "W3", "b3", "W4", "b4")]).astype(np.float32)
    m = wp.Mlp(max_batch=64)
    m.set_params(p, 1.0, 1.0)
    x = np.array([0.0, -0.0, 1e-20, 1.0, -1.0, 64.0, -64.0, 1024.0, -1e30, 2.0 ** 100], dtype=np.float32)
    X = np.zeros((x.size, 3), dtype=np.float32)
    X[:, 0] = x
    out = m.forward(dev(X.ravel())).cpu().numpy().reshape(x.size, -1)[:, 0]
    m.close()
    ref, _ = S.forward(S.from_packed(p), X.astype(np.float64), q=S.round_bf16)
    ref = ref[:, 0]
    # three bfloat16 roundings of 2^-9 at most
    assert np.all(np.abs(out - ref) <= 3 * 2.0 ** -8 * np.abs(ref) + 1e-30)
