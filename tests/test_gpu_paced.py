"""Destination-scaled FP16, two columns per lane, on a lattice whose two buffers exceed the
last-level cache (256 MiB): workgroups paced row by row and taken in alternating order.
Bitwise the state of the batched launch, which does neither, at the default strip height and
at heights that leave ragged last strips; walls at both ends and periodic."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
B = pytest.importorskip("paper_1211_6932_amd.lbmp")


@pytest.mark.parametrize("bc", [0, 1])
def test_paced_steps_are_bitwise_the_batched_ones(bc):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm device")
    nx, ny = 2502, 2803  # 2 x 140 MB; ragged in both directions
    p, (rl, rg) = W.base_params(nx, ny, t_over_tc=0.8, bc=bc), W.coexistence(0.8)
    rng = np.random.default_rng(7)
    field = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32))
    rho = field(W.droplet_field(nx, ny, 700.0, rl, rg, periodic_y=bc == 0))
    ux, uy = (field(0.01 * rng.standard_normal((ny, nx))) for _ in range(2))
    b = B.Batch([p], [rho], [ux], [uy], store="f16dest")
    b.step(5)
    for rows in (-1, 1, 6, 64):
        print(f"[gpu-case] paced {nx}x{ny} bc={bc} rows={rows}", flush=True)
        s = B.Sim(p, rho, ux, uy, store="f16dest")
        s.set_launch(strip_rows=rows)
        s.step(2).step(3)
        s.check()
        st = s.get_state()
        assert torch.equal(st, b.get_state(0, st.numel())), rows
        s.close()
    b.close()
