"""Several time steps per launch by regions of 32 x 32 sites: bitwise the same state as single
steps by strips, for every storage type and stencil, every number of steps a launch takes (1
to what the size allows), lattices smaller than a region (which then wraps around several
times), one region's tile exactly, one column more, and several ragged regions; states
carried on by the other way of stepping and through captured graphs; an unstable site is
reported."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
B = pytest.importorskip("paper_1211_6932_amd.lbmp")

KINDS = [("f32", 0), ("f32", 1), ("f16", 0), ("bf16", 0), ("f16local", 0), ("bf16local", 0), ("f16dest", 0)]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm device")
    B.load()
    yield


def lattice(nx, ny, bc, psi, stencil):
    rng = np.random.default_rng(1000 * nx + ny)
    if psi:
        p, (rl, rg) = W.ss_params(nx, ny, G=-2.7, eps=1.0, sigma=1.0 / (16 * 2.7), bc=bc), (1.6113, 0.1073)
    else:
        p, (rl, rg) = W.base_params(nx, ny, t_over_tc=0.8, bc=bc), W.coexistence(0.8)
    rho = W.droplet_field(nx, ny, 0.3 * min(nx, ny), rl, rg, periodic_y=bc == 0)
    u = 0.01 * rng.standard_normal((2, ny, nx))
    return dict(p, stencil=stencil), rl, *[torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32))
                                           for a in (rho, u[0], u[1])]


def make(case, store):
    p, rl, rho, ux, uy = case
    return B.Sim(p, rho, ux, uy, store=store, rho_ref=0.5 * rl if store in ("f16", "bf16") else 0.0)


def state(sim):
    sim.check()
    return sim.get_state().cpu().numpy()


@pytest.mark.parametrize("store,stencil", KINDS)
@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("nx,ny", [(3, 5), (18, 18), (33, 64), (61, 45), (200, 131)])
def test_regions_are_bitwise_single_steps(nx, ny, bc, store, stencil):
    for psi in (0, 1):
        print(f"[gpu-case] regions {nx}x{ny} bc={bc} psi={psi} {store} stencil={stencil}", flush=True)
        case = lattice(nx, ny, bc, psi, stencil)
        one, reg = make(case, store), make(case, store)
        one.set_launch(strip_rows=3)
        for n in range(1, 10):
            for _ in range(n):
                one.step(1)
            reg.step(n)
            assert np.array_equal(state(one), state(reg)), (psi, n)
        reg.set_launch(strip_rows=2)  # strips from here
        one.set_launch(strip_rows=-1)  # regions from here
        assert np.array_equal(state(one.step(5)), state(reg.step(5)))
        one.close(), reg.close()


@pytest.mark.parametrize("store,stencil", [("f32", 0), ("f32", 1), ("f16dest", 0)])
def test_graphs_of_region_launches(store, stencil):
    case = lattice(90, 64, 1, 0, stencil)
    a, b = make(case, store), make(case, store)
    a.set_launch(strip_rows=2)
    for _ in range(75):
        a.step(1)
    for chunk, n in ((6, 33), (2, 3), (32, 39)):
        b.set_launch(graph_chunk=chunk)
        b.step(n)
    assert np.array_equal(state(a), state(b))
    a.close(), b.close()


@pytest.mark.parametrize("bc", [0, 1])
def test_an_unstable_site_is_reported(bc):
    """A site far too dense for the equation of state (b rho / 4 >= 1) after the state was
    written: every number of steps per launch raises what single steps raise."""
    case = lattice(64, 40, bc, 0, 0)
    for n in range(1, 7):
        s = make(case, "f32")
        st = s.get_state().view(torch.float32).reshape(9, 40, 64).clone()
        st[:, 0, 63] += 10.0
        s.set_state(st.view(torch.uint8).reshape(-1), 0)
        s.step(n)
        with pytest.raises(B.LbError):
            s.check()
        s.close()


@pytest.mark.parametrize("store,stencil,nx,ny", [("f16dest", 0, 200, 161), ("f16", 0, 300, 271), ("f32", 0, 400, 301),
                                                 ("f32", 1, 800, 700), ("f16local", 0, 1200, 1001)])
def test_a_left_over_single_step_by_strips(store, stencil, nx, ny):
    """Sizes where regions take several steps per launch but leave one step to the strips."""
    case = lattice(nx, ny, 1, 0, stencil)
    one, reg = make(case, store), make(case, store)
    one.set_launch(strip_rows=4)
    for n in (1, 2, 3, 1, 7):
        assert np.array_equal(state(one.step(n)), state(reg.step(n))), n
    one.close(), reg.close()
