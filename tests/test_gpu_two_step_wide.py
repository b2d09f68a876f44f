"""Two steps per launch in workgroups of eight wavefronts (lattices of 16384 strips and more):
bitwise the states of single steps, with one-row strips, ragged three-row strips and the
automatic height, walls at both ends of the walk and periodic; and on the 8192 x 4096 splash in
the launch shape that is benchmarked, whose single step the sampled oracle test checks."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
B = pytest.importorskip("paper_1211_6932_amd.lbmp")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm device")
    B.load()
    yield


def single_steps(sim, n):
    for _ in range(n):
        sim.step(1)
    return sim


@pytest.mark.parametrize("psi", [0, 1])
@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("nx,ny,rows", [(1170, 820, 1), (2047, 1501, 3), (2901, 1666, -1)])
def test_eight_wavefronts_per_workgroup(nx, ny, rows, bc, psi):
    print(f"[gpu-case] two steps, eight waves {nx}x{ny} rows={rows} bc={bc} psi={psi}", flush=True)
    if psi:
        p, rl = W.ss_params(nx, ny, G=-2.7, eps=1.0, sigma=1.0 / (16 * 2.7), bc=bc), 1.6113
    else:
        p, rl = W.base_params(nx, ny, t_over_tc=0.8, bc=bc), W.coexistence(0.8)[0]
    gen = torch.Generator(device="cuda").manual_seed(nx + ny)
    rho = rl * (1.0 + 0.01 * torch.rand(ny, nx, device="cuda", generator=gen))
    ux, uy = (0.01 * torch.randn(ny, nx, device="cuda", generator=gen) for _ in range(2))
    one, two = B.Sim(p, rho, ux, uy), B.Sim(p, rho, ux, uy)
    two.set_launch(strip_rows=rows)
    want = single_steps(one, 7).get_state()
    two.step(4).step(3)
    assert torch.equal(two.get_state(), want)
    one.check(), two.check()
    one.close(), two.close()


def test_full_size_splash():
    print("[gpu-case] two steps, 8192x4096 splash", flush=True)
    w = W.splash(scale=4, Re=200)
    f = [torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)) for a in (w.rho0, w.ux0, w.uy0)]
    one, two = B.Sim(w.params, *f), B.Sim(w.params, *f)
    want = single_steps(one, 4).get_state()
    assert torch.equal(two.step(4).get_state(), want)
    one.check(), two.check()
    one.close(), two.close()
