"""Large D2Q9 grids without walls or force march strips of columns eight steps at
a time: the fields are bitwise those of the one-step kernel (variant GENERIC), on
sides that are no multiples of the 48 output columns or of the rows per wave,
narrow and flat grids, with one and two relaxations, with launches of fewer
steps after the strips; the sums, FP64 in another order, agree to 1e-12 of the
absolute values summed."""
import pytest
import torch

import workloads as wl
from gpu_helpers import banner, need_gpu, to_dev

pytestmark = pytest.mark.gpu

GENERIC = 1


@pytest.mark.parametrize("nx,ny", [(724, 724), (961, 1009), (1501, 1003), (7, 200000), (300000, 5),
                                   (48, 60000)])
@pytest.mark.parametrize("omega_p", [None, 1.2])
def test_strips_equal_single_steps(nx, ny, omega_p):
    L = need_gpu()
    banner(f"strips {nx}x{ny} omega_p={omega_p}")
    shape = (1, ny, nx)
    drho, u = wl.random_state(shape, 2, seed=107, du=0.03, drho=0.01)
    out = []
    for variant in (0, GENERIC):
        s = L.Solver(9, nx, ny, 1, 1.7, omega_p=omega_p, variant=variant)
        s.set_state(to_dev(drho), to_dev(u))
        s.step(19)  # two launches of eight steps, then three steps
        dr, uu = s.moments()
        out.append((dr, uu, s.diagnostics()))
        s.step(8)  # ends with the strips' own sums
        dr, uu = s.moments()
        out[-1] += (dr, uu, s.diagnostics())
        s.close()
    a, b = out
    for k in (0, 1, 3, 4):
        assert bool(torch.isfinite(a[k]).all()) and torch.equal(a[k], b[k])
    for k in (2, 5):
        assert abs(a[k][0] - b[k][0]) <= 1e-12 * (nx * ny)
        assert abs(a[k][1] - b[k][1]) <= 1e-12 * b[k][1]
