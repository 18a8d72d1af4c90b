"""Mass and energy of a step against FP64 sums of the fields it leaves, as
lwacm_moments forms them.  With a temperature on sides that are no multiples of
the tile every kernel adds node by node in FP64, so the two agree to its
rounding: 1e-12 of the absolute values summed."""
import numpy as np
import pytest
import torch

import workloads as wl
from gpu_helpers import banner, need_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(8, 17, 33), (61, 65, 63), (75, 47, 95), (64, 64, 70),
                                   (40, 33, 64)])
@pytest.mark.parametrize("walls", [False, True])
def test_sums_with_a_temperature_on_ragged_sides(shape, walls):
    L = need_gpu()
    banner(f"sums, temperature {shape} walls={walls}")
    nz, ny, nx = shape
    kw = {}
    if walls:
        m = (np.random.Generator(np.random.PCG64(191)).random(shape) < 0.03).astype(np.uint8)
        m[:, :, 0], m[:, -1] = 1, 2
        kw = dict(mask=to_dev(m, torch.uint8),
                  wall_u=[list(r) for r in wl.wall_table((0.04, 0.01, 0.0))])
    s = L.Solver(19, nx, ny, nz, 1.6, **kw)
    drho, u = wl.random_state(shape, 3, seed=193, du=0.03, drho=0.01)
    s.set_state(to_dev(drho), to_dev(u))
    s.set_thermal(1.4, to_dev(1.0 + drho), wall_T=(float("nan"), 0.9, 1.1))
    hist = torch.zeros(16, dtype=torch.float64, device="cuda")
    L.lwacm_set_diag_history(s.ctx, hist)
    s.step(3)
    dr, uu, (m0, e0) = s.moments(diagnostics=True)
    m1, e1 = s.diagnostics()
    s.close()
    n = float(np.prod(shape))
    # (the mass is the deviation plus the number of fluid nodes: one rounding)
    assert abs(m1 - m0) <= 1e-12 * float(dr.double().abs().sum()) + 2.0 ** -52 * n
    assert abs(e1 - e0) <= 1e-12 * e0
    fluid = n if not walls else float((to_dev(m, torch.uint8) == 0).sum())
    assert abs(float(hist[6]) + fluid - m1) <= 2.0 ** -52 * n and float(hist[7]) == e1
