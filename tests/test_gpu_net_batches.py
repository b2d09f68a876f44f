"""The network's two-launch passes at the batch sizes where their split changes: 16 (forward
only) and 32 rows, remainders of the gradients' steps of 128 and 512 rows, and the change from
4 to 16 rows per workgroup at 1024; buffers larger than the batch, and a smaller batch after a
larger one.  Bounds of the oracle tests of the same quantities (bf16 operand rounding on both
sides): 2e-4 forward and 1e-3 gradients, relative Frobenius; loss 1e-5."""
import numpy as np
import pytest

from oracle import mlp as M

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
B = pytest.importorskip("paper_1211_6932_amd.lbmp")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm device")
    B.load()
    yield


def inputs(n, seed):
    r = np.random.default_rng(seed)
    x = np.stack([r.choice([0.25, 0.5, 1.0], n), r.uniform(0.5, 0.85, n), r.uniform(25, 77, n), r.uniform(1, 15, n)], 1)
    base = r.uniform(-6, -0.7, (n, 128))
    return x.astype(np.float32), base.astype(np.float32), (base + 0.05 * r.standard_normal((n, 128))).astype(np.float32)


def theta32(seed):
    r = np.random.default_rng(seed)
    return (0.08 * r.standard_normal(M.N_PARAMS)).astype(np.float32)


MU, SD = np.array([0.6, 0.68, 50.0, 8.0]), np.array([0.3, 0.1, 15.0, 4.0])


def rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


def test_batches():
    th = theta32(3)
    net = B.Net(th, MU, SD, max_batch=2048)
    for n in (2048, 16, 32, 160, 544, 1024, 1056, 32):
        print(f"[gpu-case] network batch {n}", flush=True)
        x, base, t = inputs(n, n)
        z = ((x - MU.astype(np.float32)) * (1.0 / SD).astype(np.float32)).astype(np.float64)
        y, cache = M.forward(th.astype(np.float64), z, bf16=True, base=base.astype(np.float64))
        assert rel(net.forward(x, base).cpu().numpy() - base, y - base) <= 2e-4
        if n % 32:
            continue
        loss, g = net.loss_grad(x, t, base)
        want, gw = M.loss_and_grad(th.astype(np.float64), z, t.astype(np.float64), bf16=True, base=base.astype(np.float64))
        assert abs(loss / want - 1.0) <= 1e-5
        at, g = 0, g.cpu().numpy().astype(np.float64)
        for _, shape in M.SHAPES:
            size = int(np.prod(shape))
            assert rel(g[at:at + size], gw[at:at + size]) <= 1e-3, (n, shape)
            at += size
    net.close()


@pytest.mark.parametrize("batch", [32, 544])
def test_training_loop_and_single_steps_agree_bitwise(batch):
    print(f"[gpu-case] training loop batch {batch}", flush=True)
    x, base, t = (torch.from_numpy(a).cuda() for a in inputs(1500, 7))
    idx = torch.stack([torch.randperm(1500, generator=torch.Generator().manual_seed(k))[:batch] for k in range(6)])
    lr = torch.linspace(1e-3, 1e-4, 6)
    a, b = (B.Net(theta32(5), MU, SD, max_batch=1024) for _ in range(2))
    loss = torch.zeros(6, device="cuda")
    a.train_steps(x, t, idx.int().cuda(), lr.cuda(), base_all=base, loss=loss)
    for k in range(6):
        r = idx[k].cuda()
        got = b.train_step(x[r].contiguous(), t[r].contiguous(), float(lr[k]), base=base[r].contiguous())
        assert got == float(loss[k])
    assert torch.equal(a.params(), b.params())
    B.lbml_adam(a.net, 1e-4), B.lbml_adam(b.net, 1e-4)  # the last step's gradient, in both
    assert torch.equal(a.params(), b.params())
    a.close(), b.close()
