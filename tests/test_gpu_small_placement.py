"""Mass placement on lattices that one workgroup searches alone (up to 2048 sites, two per
thread) and just beyond: shift, mass and field against the oracle, and lists that mix sizes of
either kind bitwise the single calls."""
import numpy as np
import pytest

from oracle import profile as P

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
B = pytest.importorskip("paper_1211_6932_amd.lbmp")

SIZES = [(1, 1), (1023, 1), (32, 32), (41, 25), (33, 32), (45, 45), (2047, 1), (64, 32), (683, 3), (46, 45)]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm device")
    B.load()
    yield


def droplet():
    r = (np.arange(128) - 63.5) * 0.5
    return np.log(0.26 - 0.24 * np.tanh(r / 2.5)).astype(np.float32)


@pytest.mark.parametrize("nx,ny", SIZES)
def test_shift_and_mass(nx, ny):
    L, R, cx, cy = droplet(), 0.25 * min(nx, ny), 0.45 * nx, 0.55 * ny
    L64 = L.astype(np.float64)
    m0 = P.to_rho0(L64, R, cx, cy, nx, ny).sum()
    for mass in (1.002 * m0, 0.97 * m0, 100.0 * m0, 1e-3 * m0):
        print(f"[gpu-case] small placement {nx}x{ny} {mass / m0:g}", flush=True)
        field, shift = B.profile_to_rho0_mass(torch.from_numpy(L).cuda(), R, cx, cy, nx, ny, mass)
        torch.cuda.synchronize()
        d, m = shift.tolist()
        ref, delta = P.to_rho0_mass(L64, R, cx, cy, nx, ny, mass)
        assert abs(d - delta) <= 1e-9
        want = P.to_rho0(L64, R + d, cx, cy, nx, ny)
        assert abs(m - want.sum()) <= 1e-12 * want.sum()
        assert np.abs(field.cpu().numpy() / want - 1).max() < 1e-6


@pytest.mark.parametrize("sizes", [SIZES, SIZES[:8], [(200, 150), (33, 32)], [(64, 32)] * 40])
def test_lists_are_the_single_calls(sizes):
    L = torch.from_numpy(np.stack([droplet() + 0.01 * i for i in range(len(sizes))]).astype(np.float32)).cuda()
    places = [(0.25 * min(nx, ny), 0.45 * nx, 0.55 * ny, nx, ny, 0.05 * nx * ny) for nx, ny in sizes]
    print(f"[gpu-case] small placement, {len(sizes)} profiles", flush=True)
    fields, shifts = B.profiles_to_rho0_mass(L, places)
    torch.cuda.synchronize()
    for i, place in enumerate(places):
        field, shift = B.profile_to_rho0_mass(L[i], *place)
        torch.cuda.synchronize()
        assert torch.equal(field, fields[i]) and torch.equal(shift, shifts[i]), i
