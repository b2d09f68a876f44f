"""The network's own matrix products (fragment order, both directions, gradients) exactly: with
weights that permute, values that bfloat16 holds and pre-activations beyond 8, where the
activation and its derivative are exactly z and 1 in float32, every output and gradient is a
sum of a few exact products.  A lane, row or column out of place changes a value.  Rows per
workgroup 4 and 16 (batches up to and beyond 1024)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
B = pytest.importorskip("paper_1211_6932_amd.lbmp")

SIZES = [(256, 4), (256, 256), (256, 256), (128, 256)]


def bf16(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(torch.bfloat16).float().numpy()


def layers(rng):
    """(W, b) of every layer: each output of a hidden layer is one input (a permutation; a small
    integer multiple of one feature in the first), the head adds and subtracts pairs."""
    first = np.zeros((256, 4))
    first[np.arange(256), rng.integers(0, 4, 256)] = rng.integers(1, 4, 256)
    second, third = (np.eye(256)[rng.permutation(256)] for _ in range(2))
    head = np.zeros((128, 256))
    pairs = rng.permutation(256).reshape(128, 2)
    head[np.arange(128), pairs[:, 0]], head[np.arange(128), pairs[:, 1]] = 1.0, -2.0
    bias = [rng.integers(8, 100, 256), np.zeros(256), np.zeros(256), rng.integers(-20, 20, 128)]
    return list(zip((first, second, third, head), bias))


@pytest.mark.parametrize("n", [32, 160, 1024, 1056])
def test_exact_products(n):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm device")
    print(f"[gpu-case] network layout B={n}", flush=True)
    rng = np.random.default_rng(n)
    net_layers = layers(rng)
    theta = np.concatenate([np.concatenate([w.reshape(-1), b]) for w, b in net_layers]).astype(np.float32)
    assert theta.size == B.LBML_PARAMS
    x = rng.integers(0, 8, (n, 4)).astype(np.float64)
    acts, h = [x], x
    for i, (w, b) in enumerate(net_layers):
        h = h @ w.T + b
        if i < 3:
            assert h.min() >= 8 and np.array_equal(bf16(h), h)
            acts.append(h)
    net = B.Net(theta, [0.0] * 4, [1.0] * 4, max_batch=n)
    got = net.forward(torch.from_numpy(x.astype(np.float32))).cpu().numpy()
    assert np.array_equal(got, h)
    # targets at integer distances: dY = 2 d / (128 n) is d times an exact bfloat16 only for a power
    # of two, so the exact gradient takes the rounded one on
    d = rng.integers(-3, 4, (n, 128)).astype(np.float64)
    loss, grad = net.loss_grad(torch.from_numpy(x.astype(np.float32)), torch.from_numpy((h - d).astype(np.float32)))
    assert abs(loss / (d * d).mean() - 1.0) <= 1e-6
    dz = bf16(np.float32(2.0 / (128.0 * n)) * d.astype(np.float32)).astype(np.float64)
    want, most = [], 0.0  # most: largest |dz| of any layer
    for i in range(3, -1, -1):
        w, _ = net_layers[i]
        most = max(most, np.abs(dz).max())
        want = [(dz.T @ acts[i]).reshape(-1), dz.sum(0)] + want
        if i:
            dz = bf16(dz @ w).astype(np.float64)
    want, grad = np.concatenate(want), grad.cpu().numpy().astype(np.float64)
    # sums of n products that FP32 holds, added in FP32: at most n roundings of 2^-24 of the sum of
    # their magnitudes; at powers of two (n = 32, 1024) dz has few bits and nothing is rounded
    exact = n & (n - 1) == 0
    bound = 0.0 if exact else n * 2.0 ** -24 * n * max(a.max() for a in acts) * most
    assert np.abs(grad - want).max() <= bound
    net.close()
