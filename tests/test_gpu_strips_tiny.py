"""The strip kernels of the 16-bit encodings on the smallest and ragged grids, which the automatic
choice leaves to regions: one step from the same stored state is the oracle's, rounded once
(the bound of the precision tests).  Even widths run the two-columns-per-lane step for f16dest:
4 (smallest), 126 (a full 124-column tile and a 2-column one), 248 (two full tiles)."""
import numpy as np
import pytest

import test_gpu_precision as TP
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not TP.torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm device")
    TP.B.load()
    yield


@pytest.mark.parametrize("store", TP.GLOBAL + TP.LOCAL + TP.DEST)
@pytest.mark.parametrize("shape", [(3, 3), (5, 3), (3, 70), (64, 3), (63, 125), (3, 4), (5, 6), (4, 126), (7, 248),
                                   (9, 124), (40, 130)])
def test_one_step_by_strips(store, shape):
    ny, nx = shape
    rho0 = 0.2 + 0.02 * np.random.default_rng(nx * 1000 + ny).standard_normal((ny, nx))
    for bc in (0, 1):
        p = W.base_params(nx, ny, a=0.5, t_over_tc=0.8, bc=bc)
        w = W.Workload("tiny", p, rho0, info=dict(rho_l=0.2))
        for rows in (1, 3, 8):
            print(f"[gpu-case] strips one-step store={store} shape={shape} bc={bc} rows={rows}", flush=True)
            excess = TP.one_step_excess(w, store, strip_rows=rows)
            assert excess <= 0.0, (store, shape, bc, rows, excess)
