"""Moments and diagnostics passes at the edges of their strips and tiles: the diagnostics'
sums equal FP64 sums over the moments' fields (both passes evaluate the same FP32 density
and velocity per site; a sum of n terms in another order differs by at most n 2^-53 of the
sum of magnitudes), for both stencils, and a batch's diagnostics in one call equal those of
the lattices alone, with an unstable lattice among them."""
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


def f32(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32))


@pytest.mark.parametrize("stencil", [0, 1])
@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("nx,ny", [(3, 3), (60, 4), (61, 5), (62, 7), (63, 33), (125, 9), (2100, 1030)])
def test_diagnostics_sum_the_moments(nx, ny, bc, stencil):
    print(f"[gpu-case] passes {nx}x{ny} bc={bc} stencil={stencil}", flush=True)
    p = dict(W.base_params(nx, ny, t_over_tc=0.8, bc=bc), stencil=stencil)
    rl, rg = W.coexistence(0.8)
    rho0 = W.droplet_field(nx, ny, 0.3 * min(nx, ny), rl, rg, periodic_y=bc == 0)
    s = B.Sim(p, f32(rho0), f32(np.full((ny, nx), 0.01)), f32(np.full((ny, nx), -0.02)))
    s.step(3)
    rho, ux, uy = (t.cpu().numpy().astype(np.float64) for t in s.moments())
    d = s.diagnostics(0.5 * nx, 0.5 * ny, 2.5, 2.5)
    s.close()
    n = nx * ny
    for got, v in ((d["mass"], rho), (d["mom_x"], rho * ux), (d["mom_y"], rho * uy)):
        assert abs(got - v.sum()) <= 2 * n * 2.0 ** -53 * np.abs(v).sum()
    assert d["n_in"] + d["n_out"] == n
    speed = np.sqrt((ux * ux + uy * uy).astype(np.float32).astype(np.float64)).max()
    assert abs(d["max_u"] - speed) <= 1e-6 * speed


def test_batch_diagnostics_with_an_unstable_lattice():
    """The original forcing at T/T_c = 0.6 goes unstable; the lattices beside it are reported
    as alone, before and after it has been flagged."""
    ws = [W.stationary_droplet(n=64, R0=14), W.stationary_droplet(n=96, R0=24, sigma=0.0, nu_l=0.0334, nu_g=0.0334),
          W.stationary_droplet(n=67, R0=15)]
    print("[gpu-case] batch diagnostics with an unstable lattice", flush=True)
    b = B.Batch([w.params for w in ws], [f32(w.rho0) for w in ws])
    b.step(3000)
    rin = [(31.5, 31.5, 0.0, 7.0)] * 3
    rout = [(31.5, 31.5, 25.0, float("inf"))] * 3
    first = b.diagnostics_all(rin, rout)
    again = b.diagnostics_all(rin, rout)
    assert [d["unstable"] for d in first] == [0, 1, 0] and [d["unstable"] for d in again] == [0, 1, 0]
    assert again[1]["mass"] == 0.0 and first[0] == again[0] and first[2] == again[2]
    assert b.check() == (B.LB_EUNSTABLE, 1)
    for i in (0, 2):
        s = B.Sim(ws[i].params, f32(ws[i].rho0))
        s.step(3000)
        assert s.diagnostics(31.5, 31.5, 7.0, 25.0) == first[i]
        s.close()
    b.close()
