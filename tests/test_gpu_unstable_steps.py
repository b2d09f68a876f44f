"""A site that becomes invalid one step after a valid state: a velocity far beyond the lattice's
range keeps the site's own density and drives its neighbours' out of bounds one step later (the
oracle takes the first step and refuses the second).  One step reports nothing, two steps in
one call report it, whether a launch takes both (strips of two steps, regions, batches) or one
each; for sites next to the columns and rows where the launches divide the lattice."""
import numpy as np
import pytest

import workloads as W
from oracle import lbref as O

torch = pytest.importorskip("torch")
B = pytest.importorskip("paper_1211_6932_amd.lbmp")

NX, NY = 130, 70
SPIKE = 2.0
# columns of the 58- and 62-column strips and of the regions' tiles (26 wide for two steps of the
# nearest-neighbour stencil, 22 for 24 sites), rows of the strips and regions, walls and corners
SITES = [(0, 0), (129, 69), (57, 20), (58, 21), (59, 8), (61, 22), (62, 26), (25, 25), (26, 27), (21, 43), (22, 44),
         (115, 35), (116, 69), (129, 0), (3, 34), (64, 52)]


def case(bc, site, store="f32", stencil=0, psi=0):
    if psi:
        p, rl = W.ss_params(NX, NY, G=-2.7, eps=1.0, sigma=1.0 / (16 * 2.7), bc=bc), 1.6113
    else:
        p, rl = W.base_params(NX, NY, t_over_tc=0.8, bc=bc), W.coexistence(0.8)[0]
    rho, ux = np.full((NY, NX), rl, dtype=np.float32), np.zeros((NY, NX), dtype=np.float32)
    if site is not None:
        ux[site[1], site[0]] = SPIKE
    return dict(p, stencil=stencil), rho, ux, np.zeros_like(ux), (0.5 * rl if store in ("f16", "bf16") else 0.0)


@pytest.mark.parametrize("psi,stencil", [(0, 0), (1, 0), (0, 1)])
@pytest.mark.parametrize("bc", [0, 1])
def test_the_oracle_refuses_the_second_step(bc, psi, stencil):
    for site in SITES:
        p, rho, ux, uy, _ = case(bc, site, stencil=stencil, psi=psi)
        s = O.State(O.Params(**p), rho.astype(np.float64), ux.astype(np.float64), uy.astype(np.float64))
        s.step(1)
        with pytest.raises(O.OracleError):
            s.step(1)


def sim(bc, site, store, stencil, psi, rows):
    p, rho, ux, uy, ref = case(bc, site, store, stencil, psi)
    s = B.Sim(p, *[torch.from_numpy(a) for a in (rho, ux, uy)], store=store, rho_ref=ref)
    if rows:
        s.set_launch(strip_rows=rows)
    return s


@pytest.mark.gpu
@pytest.mark.parametrize("store,stencil,psi,rows", [
    ("f32", 0, 0, 0), ("f32", 0, 1, 0), ("f32", 0, 0, 5), ("f32", 0, 1, 1), ("f32", 0, 0, 64), ("f32", 1, 0, 0),
    ("f32", 1, 0, 4), ("f16", 0, 0, 0), ("bf16", 0, 0, 4), ("f16local", 0, 0, 0), ("f16local", 0, 0, 3),
    ("f16dest", 0, 0, 0), ("f16dest", 0, 0, 5)])
@pytest.mark.parametrize("bc", [0, 1])
def test_single_lattices(bc, store, stencil, psi, rows):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm device")
    for site in SITES:
        print(f"[gpu-case] unstable second step {store} stencil={stencil} psi={psi} rows={rows} bc={bc} {site}", flush=True)
        s = sim(bc, site, store, stencil, psi, rows)
        s.step(1)
        s.check()
        s.step(1)
        with pytest.raises(B.LbError):
            s.check()
        s.close()
        s = sim(bc, site, store, stencil, psi, rows)
        s.step(2)
        with pytest.raises(B.LbError):
            s.check()
        s.close()


@pytest.mark.gpu
@pytest.mark.parametrize("store", ["f32", "f16local", "f16dest"])
@pytest.mark.parametrize("bc", [0, 1])
def test_batches(bc, store):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm device")
    for rows in (0, 1, 5):
        print(f"[gpu-case] unstable second step, batch {store} rows={rows} bc={bc}", flush=True)
        for n in (1, 2):
            lattices = [case(bc, site, store) for site in SITES] + [case(bc, None, store)]
            b = B.Batch([c[0] for c in lattices], *[[torch.from_numpy(c[k]) for c in lattices] for k in (1, 2, 3)], store=store)
            if rows:
                b.set_launch(B.LB_BATCH_STEPWISE, rows)
            b.step(n)
            assert b.check() == ((B.LB_OK, 0) if n == 1 else (B.LB_EUNSTABLE, len(SITES)))
            b.close()
