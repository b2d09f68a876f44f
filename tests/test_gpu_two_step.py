"""Two time steps per launch (FP32, nearest-neighbour stencil): bitwise the same state as
single steps, at the edges of its 58-column tiles, the smallest lattices, ragged strips
of every height class (walls at both ends of one strip, strips off the walls, both walk
directions) and both pseudopotential forms."""
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


def lattice(nx, ny, bc, psi=0):
    rng = np.random.default_rng(1000 * nx + ny)
    if psi:
        p, (rl, rg) = W.ss_params(nx, ny, G=-2.7, eps=1.0, sigma=1.0 / (16 * 2.7), bc=bc), (1.6113, 0.1073)
    else:
        p, (rl, rg) = W.base_params(nx, ny, t_over_tc=0.7, bc=bc), W.coexistence(0.7)
    rho = W.droplet_field(nx, ny, 0.3 * min(nx, ny), rl, rg, periodic_y=bc == 0)
    u = 0.01 * rng.standard_normal((2, ny, nx))
    return p, *[torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)) for a in (rho, u[0], u[1])]


def state(sim):
    sim.check()
    return sim.get_state().cpu().numpy()


@pytest.mark.parametrize("psi", [0, 1])
@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("nx,ny", [(8, 8), (57, 9), (58, 31), (59, 40), (117, 12), (174, 65), (700, 130)])
def test_two_steps_per_launch_are_bitwise_single_steps(nx, ny, bc, psi):
    p, rho, ux, uy = lattice(nx, ny, bc, psi)
    one = B.Sim(p, rho, ux, uy)
    for _ in range(11):
        one.step(1)
    ref = state(one)
    one.close()
    for rows in (-1, 1, 2, 3, 7, 64):
        print(f"[gpu-case] two steps per launch {nx}x{ny} bc={bc} psi={psi} rows={rows}", flush=True)
        s = B.Sim(p, rho, ux, uy)
        s.set_launch(strip_rows=rows)
        s.step(4).step(7)
        assert s.t == 11
        assert np.array_equal(state(s), ref), rows
        s.close()


@pytest.mark.parametrize("chunk", [2, 6, 32])
def test_graphs_of_any_even_length_end_in_the_right_buffer(chunk):
    p, rho, ux, uy = lattice(130, 90, 1)
    a, b = B.Sim(p, rho, ux, uy), B.Sim(p, rho, ux, uy)
    for _ in range(75):
        a.step(1)
    b.set_launch(graph_chunk=chunk)
    b.step(33).step(3).step(39)
    assert np.array_equal(state(a), state(b))
    a.close(), b.close()


@pytest.mark.parametrize("bc", [0, 1])
def test_batch_two_steps_per_launch(bc):
    """Lattices of 8 to 174 columns in one batch, odd and even step counts across calls and a
    captured graph, default and fixed heights, against single steps of each lattice alone; a
    batch with a lattice below 8 x 8 (stepped one at a time) gives the same states."""
    sizes = [(8, 8), (58, 9), (174, 65), (61, 40)]
    ls = [lattice(nx, ny, bc) for nx, ny in sizes]
    refs = []
    for p, rho, ux, uy in ls:
        s = B.Sim(p, rho, ux, uy)
        for _ in range(42):
            s.step(1)
        refs.append(state(s))
        s.close()
    for rows, extra in ((0, False), (1, False), (5, False), (64, False), (0, True)):
        print(f"[gpu-case] batch two steps bc={bc} rows={rows} small={extra}", flush=True)
        more = [lattice(7, 7, bc)] if extra else []
        b = B.Batch([l[0] for l in ls + more], [l[1] for l in ls + more], [l[2] for l in ls + more],
                    [l[3] for l in ls + more])
        if rows:
            b.set_launch(B.LB_BATCH_STEPWISE, rows)
        b.step(3).step(4).step(35)
        assert b.check() == (B.LB_OK, 0)
        for i, (l, ref) in enumerate(zip(ls, refs)):
            assert np.array_equal(b.get_state(i, B.lb_state_bytes(B.make_params(l[0], "f32"))).cpu().numpy(), ref), (rows, i)
        b.close()
