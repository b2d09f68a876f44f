"""Tensors made or used on the caller's stream: what the library reads is ordered after the work
that makes it, also where that work is still queued when the call is made, and what it writes
after work that still uses the same memory (a tensor freed a moment ago on the caller's
stream).  The queued work is held back by a long wait on that stream."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
B = pytest.importorskip("paper_1211_6932_amd.lbmp")

NX, NY = 256, 192
WAIT = 100_000_000  # clock cycles: tens of milliseconds


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm device")
    B.load()
    yield


@pytest.fixture(params=["default", "side"])
def caller(request):
    """The caller's stream: torch's default one, or another."""
    s = torch.cuda.current_stream() if request.param == "default" else torch.cuda.Stream()
    with torch.cuda.stream(s):
        yield s
    torch.cuda.synchronize()


def fields():
    p, (rl, rg) = W.base_params(NX, NY, t_over_tc=0.8), W.coexistence(0.8)
    rho = torch.from_numpy(W.droplet_field(NX, NY, 40.0, rl, rg).astype(np.float32)).cuda()
    flat = torch.full_like(rho, rl)
    torch.cuda.synchronize()
    return p, rho, flat


def late(now, then):
    """A tensor holding `now` until queued work has written `then` into it."""
    t = now.clone()
    torch.cuda.current_stream().synchronize()
    torch.cuda._sleep(WAIT)
    t.copy_(then)
    return t


def test_lattice_inputs(caller):
    print("[gpu-case] stream order: inputs of a lattice", flush=True)
    p, rho, flat = fields()
    sim = B.Sim(p, late(flat, rho))
    assert torch.equal(sim.moments()[0], B.Sim(p, rho).moments()[0])
    batch = B.Batch([p, p], [late(flat, rho), rho])
    assert torch.equal(batch.moments(0)[0], batch.moments(1)[0])
    sim.step(3)
    other = B.Sim(p, flat)
    other.set_state(late(other.get_state(), sim.get_state()), 3)
    assert torch.equal(other.get_state(), sim.get_state())


def test_network_inputs(caller):
    print("[gpu-case] stream order: inputs of the network", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(1)
    theta = 0.08 * torch.randn(B.LBML_PARAMS, device="cuda", generator=gen)
    x, t = torch.rand(32, 4, device="cuda", generator=gen), torch.randn(32, 128, device="cuda", generator=gen)
    torch.cuda.synchronize()
    mu, sd = [0.0] * 4, [1.0] * 4
    a, b = B.Net(theta, mu, sd, max_batch=32), B.Net(late(torch.zeros_like(theta), theta), mu, sd, max_batch=32)
    assert torch.equal(b.params(), theta)
    b.set_params(late(torch.zeros_like(theta), theta))
    assert torch.equal(b.params(), theta)
    assert a.train_step(x, t, 1e-3) == b.train_step(late(torch.zeros_like(x), x), late(torch.zeros_like(t), t), 1e-3)
    assert torch.equal(a.params(), b.params())
    a.close(), b.close()


def test_outputs_in_memory_still_in_use(caller):
    print("[gpu-case] stream order: outputs", flush=True)
    p, rho, _ = fields()
    sim, batch = B.Sim(p, rho), B.Batch([p, p], [rho, rho])
    net = B.Net(torch.zeros(B.LBML_PARAMS), [0.0] * 4, [1.0] * 4, max_batch=32)
    for call in (lambda: sim.moments(), lambda: [sim.get_state()], lambda: batch.moments(1),
                 lambda: [batch.get_state(0, B.lb_state_bytes(sim.p))], lambda: [net.params()]):
        want = [o.clone() for o in call()]
        blocks = call()  # of the very sizes, so that the next call's outputs fall into them
        torch.cuda.current_stream().synchronize()
        torch.cuda._sleep(WAIT)
        for o in blocks:
            o.fill_(7)
        del blocks, o
        got = call()
        torch.cuda.synchronize()
        assert all(torch.equal(g, w) for g, w in zip(got, want))


def test_learned_starts(caller, monkeypatch):
    """Prediction and placement are on one stream, the caller's."""
    from paper_1211_6932_amd import initialiser as I
    print("[gpu-case] stream order: learned starts", flush=True)
    ws = [W.stationary_droplet(n=96, R0=20 + i) for i in range(3)]
    for w in ws:
        w.info.update(cx=47.5, cy=47.5)
    r = torch.arange(128, device="cuda") * 0.5 - 31.75
    prof = torch.log(0.26 - 0.24 * torch.tanh(r / 2.5)).repeat(3, 1)
    torch.cuda.synchronize()
    monkeypatch.setattr(I, "predict", lambda model, w, anchored=True: prof)
    want = I.learned_rho0(None, ws)
    monkeypatch.setattr(I, "predict", lambda model, w, anchored=True: late(torch.zeros_like(prof), prof))
    got = I.learned_rho0(None, ws)
    assert got[1] == want[1] and all(torch.equal(a, b) for a, b in zip(got[0], want[0]))


def test_while_the_caller_captures():
    """A call on the library's own stream while the caller's stream is being captured neither joins
    nor breaks the capture."""
    print("[gpu-case] stream order: capture", flush=True)
    p, rho, _ = fields()
    sim = B.Sim(p, rho)
    want = sim.moments()
    x = torch.ones(8, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, capture_error_mode="relaxed"):
        y = x + 1.0
        got = sim.step(0).moments()
    g.replay()
    torch.cuda.synchronize()
    assert bool((y == 2.0).all()) and all(torch.equal(a, b) for a, b in zip(got, want))
