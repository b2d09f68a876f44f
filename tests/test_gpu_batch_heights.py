"""Heights and workgroup sizes of the two-step launches of a batch: a few lattices (every strip
resident, 4 wavefronts per workgroup) and enough one-row strips for workgroups of 8 spanning
several lattices, automatic and fixed heights, heights that do not divide the lattices:
bitwise the single steps of each lattice alone."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
B = pytest.importorskip("paper_1211_6932_amd.lbmp")


@pytest.mark.parametrize("n", [3, 96])
@pytest.mark.parametrize("bc", [0, 1])
def test_batch_heights_are_bitwise_single_steps(n, bc):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm device")
    rng = np.random.default_rng(n)
    rl, rg = W.coexistence(0.8)
    ps, rhos = [], []
    for i in range(n):  # 96: about 96 x 2 x 45 one-row strips, more than 16 per compute unit
        nx, ny = int(rng.integers(40, 140)), int(rng.integers(8, 90))
        ps.append(W.base_params(nx, ny, t_over_tc=0.8, bc=bc))
        rho = W.droplet_field(nx, ny, 0.3 * min(nx, ny), rl, rg, periodic_y=bc == 0)
        rhos.append(torch.from_numpy(np.ascontiguousarray(rho, dtype=np.float32)))
    refs = {}
    for i in (0, 1, n // 2, n - 1):
        s = B.Sim(ps[i], rhos[i])
        s.set_launch(strip_rows=3)
        for _ in range(7):
            s.step(1)
        refs[i] = s.get_state()
        s.close()
    for rows in (0, 1, 5, 16):
        print(f"[gpu-case] batch of {n} bc={bc} rows={rows}", flush=True)
        b = B.Batch(ps, rhos)
        b.set_launch(0, rows)
        b.step(4).step(3)
        for i, ref in refs.items():
            assert torch.equal(b.get_state(i, ref.numel()), ref), (rows, i)
        b.close()
