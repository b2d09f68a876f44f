"""Profile fit and mass placement where their splits change: rows of one chunk of 256 sites
more or less, an odd number of rows, lattices up to and beyond the 1024 sites that one
workgroup searches alone, fields that are not 8-byte aligned, profiles whose mass does not
grow monotonically, and masses out of reach; against the oracle (FP64 on both sides, sums in
another order, FP32 output)."""
import numpy as np
import pytest

import workloads as W
from oracle import profile as P

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
B = pytest.importorskip("paper_1211_6932_amd.lbmp")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm device")
    B.load()
    yield


@pytest.mark.parametrize("nx,ny", [(2, 2), (255, 3), (256, 17), (257, 64), (513, 130), (40, 301)])
def test_extract(nx, ny):
    print(f"[gpu-case] profile extract {nx}x{ny}", flush=True)
    rng = np.random.default_rng(nx + ny)
    R = 0.3 * min(nx, ny)
    rho = (W.droplet_field(nx, ny, R, 0.3, 0.01) * np.exp(0.01 * rng.standard_normal((ny, nx)))).astype(np.float32)
    got = B.profile_extract(torch.from_numpy(rho).cuda(), 0.4 * nx, 0.6 * ny, R).cpu().numpy()
    ref = P.extract(rho.astype(np.float64), 0.4 * nx, 0.6 * ny, R)
    # the bound of the fit's oracle test: rounding to FP32 and the condition of the samples
    # that few sites reach
    assert np.abs(got - ref).max() <= 2e-6 * max(1.0, np.abs(ref).max())


def profile(kind):
    r = (np.arange(128) - 63.5) * 0.5
    if kind == "wave":  # the mass first falls, then grows with the shift
        return (np.log(0.2) + 0.3 * np.sin(r / 4.0)).astype(np.float32)
    return np.log(0.26 - 0.24 * np.tanh(r / 2.5)).astype(np.float32)


@pytest.mark.parametrize("kind", ["droplet", "wave"])
@pytest.mark.parametrize("nx,ny", [(1, 1), (16, 16), (32, 32), (41, 25), (64, 63), (256, 257), (700, 400)])
def test_mass(nx, ny, kind):
    L, R = profile(kind), 0.25 * min(nx, ny)
    dev, cx, cy = torch.from_numpy(L).cuda(), 0.45 * nx, 0.55 * ny
    L64 = L.astype(np.float64)
    m0 = P.to_rho0(L64, R, cx, cy, nx, ny).sum()
    for mass in (1.002 * m0, 0.97 * m0, 100.0 * m0, 1e-3 * m0):
        print(f"[gpu-case] mass placement {kind} {nx}x{ny} {mass / m0:g}", flush=True)
        store = torch.full((ny * nx + 2,), -1.0, device="cuda")
        field = store[1:1 + ny * nx].reshape(ny, nx)  # 4-byte aligned only
        _, shift = B.profile_to_rho0_mass(dev, R, cx, cy, nx, ny, mass, out=field)
        torch.cuda.synchronize()
        d, m = shift.tolist()
        ref, delta = P.to_rho0_mass(L64, R, cx, cy, nx, ny, mass)
        if kind == "droplet" or not abs(delta) < 7.9:
            assert abs(d - delta) <= 1e-9
        want = P.to_rho0(L64, R + d, cx, cy, nx, ny)  # where sums tie, the mass decides, not the shift
        assert abs(m - want.sum()) <= 1e-12 * want.sum()
        assert abs(m - ref.sum()) <= 1e-9 * ref.sum()
        assert np.abs(field.cpu().numpy() / want - 1).max() < 1e-6
        assert store[0] == -1.0 and store[-1] == -1.0


def test_mass_of_many_profiles():
    """More profiles than one launch serves, of different sizes (among them lattices searched
    by one workgroup): bitwise the fields and shifts of single calls."""
    rng = np.random.default_rng(5)
    sizes = [(int(a), int(b)) for a, b in rng.integers(20, 200, (33, 2))] + [(16, 16), (32, 32), (256, 257)]
    L = torch.from_numpy(np.stack([profile("droplet") + 0.01 * i for i in range(len(sizes))]).astype(np.float32)).cuda()
    places = [(0.25 * min(nx, ny), 0.45 * nx, 0.55 * ny, nx, ny, 0.05 * nx * ny) for nx, ny in sizes]
    print("[gpu-case] mass placement of many profiles", flush=True)
    fields, shifts = B.profiles_to_rho0_mass(L, places)
    torch.cuda.synchronize()
    for i, (R, cx, cy, nx, ny, mass) in enumerate(places):
        field, shift = B.profile_to_rho0_mass(L[i], R, cx, cy, nx, ny, mass)
        torch.cuda.synchronize()
        assert torch.equal(field, fields[i]) and torch.equal(shift, shifts[i]), i


def test_fits_of_many_fields():
    """More fields than one launch serves, of different sizes: bitwise the fits of single calls."""
    rng = np.random.default_rng(6)
    sizes = [(int(a), int(b)) for a, b in rng.integers(2, 150, (34, 2))] + [(300, 257)]
    rhos = [torch.from_numpy((0.1 + rng.random((ny, nx))).astype(np.float32)).cuda() for nx, ny in sizes]
    places = [(0.4 * nx, 0.6 * ny, 0.3 * min(nx, ny)) for nx, ny in sizes]
    out = torch.full((len(sizes) + 1, 128), -1.0, device="cuda")
    each = max(B.lbml_profile_scratch_bytes(ny) for _, ny in sizes)
    scratch = torch.empty(each * len(sizes), dtype=torch.uint8, device="cuda")
    print("[gpu-case] profile fits of many fields", flush=True)
    B.profiles_extract(rhos, places, out[:len(sizes)], scratch)
    torch.cuda.synchronize()
    for i, rho in enumerate(rhos):
        assert torch.equal(B.profile_extract(rho, *places[i]), out[i]), i
    assert bool((out[-1] == -1.0).all())
    with pytest.raises(ValueError):
        B.profiles_extract(rhos, places, out[:len(sizes)], scratch[:-1])
