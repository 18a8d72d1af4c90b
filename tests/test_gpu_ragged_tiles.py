"""A temperature on D3Q19 grids whose sides are no multiples of the 32 x 16 tile
runs in the flow's tile kernel, the last tile of a side moved back to end at
it.  Against the gather kernels (variant GENERIC) on sides one more and one
less than a multiple and at the smallest sides: fields within 1e-6 after 4
steps (the bound of the other comparisons of the two), mass and energy counted once per node; and what the tile variants refuse on such
grids stays refused."""
import numpy as np
import pytest
import torch

import workloads as wl
from gpu_helpers import banner, need_gpu, rel_l2, to_dev

pytestmark = pytest.mark.gpu

GENERIC = 1


def _run(L, shape, walls, variant):
    nz, ny, nx = shape
    kw = {}
    if walls:
        m = (np.random.Generator(np.random.PCG64(101)).random(shape) < 0.03).astype(np.uint8)
        m[:, :, 0], m[:, -1] = 1, 2
        kw = dict(mask=to_dev(m, torch.uint8),
                  wall_u=[list(r) for r in wl.wall_table((0.04, 0.01, 0.0))])
    s = L.Solver(19, nx, ny, nz, 1.6, variant=variant, **kw)
    drho, u = wl.random_state(shape, 3, seed=103, du=0.03, drho=0.01)
    s.set_state(to_dev(drho), to_dev(u))
    s.set_thermal(1.4, to_dev(1.0 + drho), wall_T=(float("nan"), 0.9, 1.1))
    s.step(4)
    dr, uu, diag = s.moments(diagnostics=True)
    out = [t.double().cpu().numpy() for t in (dr, uu, s.temperature())] + [diag, s.diagnostics()]
    s.close()
    return out


@pytest.mark.parametrize("shape", [(8, 17, 33), (61, 65, 63), (75, 47, 95), (64, 64, 70)])
@pytest.mark.parametrize("walls", [False, True])
def test_temperature_on_ragged_sides(shape, walls):
    L = need_gpu()
    banner(f"ragged thermal {shape} walls={walls}")
    a, b = _run(L, shape, walls, 0), _run(L, shape, walls, GENERIC)
    for x, y in zip(a[:3], b[:3]):
        assert rel_l2(x, y) < 1e-6
    # the step's sums (FP32 per thread, each node once) against those of the fields
    (m0, e0), (m1, e1) = a[3], a[4]
    assert abs(m1 - m0) <= 2e-6 * np.abs(a[0]).sum() + 1e-9 * np.prod(shape)
    assert abs(e1 - e0) <= 2e-6 * e0


def test_tile_variants_still_refuse_ragged_sides():
    L = need_gpu()
    s = L.Solver(19, 70, 64, 64, 1.7)
    s.set_state(torch.zeros((64, 64, 70)), torch.zeros((3, 64, 64, 70)))
    for call in (lambda: L.lwacm_set_variant(s.ctx, 2), lambda: L.lwacm_set_variant(s.ctx, 3),
                 lambda: L.lwacm_set_march_chunk(s.ctx, 64)):
        with pytest.raises(L.LWACMError) as e:
            call()
        assert e.value.code == L.LWACM_EUNSUPPORTED
    st = s.save_state()
    mu = torch.zeros((64, 64, 70, 4), device="cuda")
    dw = torch.zeros(1, dtype=torch.float64, device="cuda")
    assert not L.lwacm_adjoint_step2(s.ctx, st, st, mu, torch.empty_like(mu), dw, False)
    s.close()
