"""Single steps of lattices whose two buffers exceed the last-level cache (256 MiB): every other
launch takes the workgroups in descending order.  Bitwise the states of launches that all
ascend (a state written back puts the next launch at the first buffer again), for the
one-column kernels of every storage type, odd widths and ragged strips, walls and periodic."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
B = pytest.importorskip("paper_1211_6932_amd.lbmp")


@pytest.mark.parametrize("store,nx,ny", [("f32", 2003, 1901), ("f16", 2907, 2603), ("bf16", 2907, 2603),
                                         ("f16local", 2501, 2503), ("bf16local", 2501, 2503), ("f16dest", 2701, 2503)])
@pytest.mark.parametrize("bc", [0, 1])
def test_descending_launches_are_bitwise_ascending_ones(store, nx, ny, bc):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm device")
    print(f"[gpu-case] alternating order {store} {nx}x{ny} bc={bc}", flush=True)
    p, (rl, _) = W.base_params(nx, ny, t_over_tc=0.8, bc=bc), W.coexistence(0.8)
    gen = torch.Generator(device="cuda").manual_seed(nx)
    rho = rl * (1.0 + 0.01 * torch.rand(ny, nx, device="cuda", generator=gen))
    torch.cuda.synchronize()
    a, b = (B.Sim(p, rho, store=store, rho_ref=0.5 * rl if store in ("f16", "bf16") else 0.0) for _ in range(2))
    for k in range(1, 5):
        a.step(1)
        b.step(1)
        st = b.get_state()
        assert torch.equal(a.get_state(), st), k
        b.set_state(st, k)
    a.check(), b.check()
    a.close(), b.close()
