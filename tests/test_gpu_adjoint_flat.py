"""Reverse steps on grids of fewer than eight planes whose other sides are
multiples of the tile: they run on the reverse tile kernel, with and without
walls.  Against the one-thread-per-node kernel (variant GENERIC): mu within 1e-6,
dL/domega within 1e-5 of the absolute terms summed (the bounds of the other
comparisons of the two), and not the same bits, which would be that kernel itself."""
import numpy as np
import pytest
import torch

import workloads as wl
from gpu_helpers import banner, need_gpu, rel_l2, to_dev

pytestmark = pytest.mark.gpu

GENERIC = 1


@pytest.mark.parametrize("nz", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("kind", ["plain", "walls", "fp16"])
@pytest.mark.parametrize("t0", [0, 5])
def test_flat_grids_run_the_reverse_tile_kernel(nz, kind, t0):
    L = need_gpu()
    ny, nx = 32, 64
    shape = (nz, ny, nx)
    banner(f"reverse, flat grid nz={nz} {kind} t0={t0}")
    kw = {}
    if kind == "walls":
        m = (np.random.Generator(np.random.PCG64(211)).random(shape) < 0.05).astype(np.uint8)
        m[:, 0], m[:, -1] = 1, 2
        kw = dict(mask=to_dev(m, torch.uint8),
                  wall_u=[list(r) for r in wl.wall_table((0.04, 0.01, 0.0))])
    drho, u = wl.random_state(shape, 3, seed=213, du=0.03, drho=0.01)
    s = L.Solver(19, nx, ny, nz, 1.6, storage=1 if kind == "fp16" else 0, **kw)
    s.set_state(to_dev(drho), to_dev(u))
    st = []
    for _ in range(3):
        st.append(s.save_state())
        s.step(1)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(215)
    lam = torch.randn((4,) + shape, device="cuda", generator=gen)
    seed = torch.empty(shape + (4,), device="cuda")
    L.lwacm_adjoint_seed(s.ctx, s.save_state(), lam, seed)
    out = []
    for variant in (0, GENERIC):
        L.lwacm_set_variant(s.ctx, variant)
        mu, tmp = seed.clone(), torch.empty_like(seed)
        dw = torch.zeros(1, dtype=torch.float64, device="cuda")
        for j in (2, 1, 0):
            L.lwacm_adjoint_step(s.ctx, st[j], mu, tmp, dw, t0 + j == 0)
            mu, tmp = tmp, mu
        sw, dws = seed.clone(), torch.zeros(1, dtype=torch.float64, device="cuda")
        L.lwacm_adjoint_sweep(s.ctx, torch.cat(st), t0, 3, sw, torch.empty_like(sw), dws)
        assert torch.equal(mu, sw) and float(dw) == float(dws)
        out.append((mu, float(dw)))
    s.close()
    (a, wa), (b, wb) = out
    assert bool(torch.isfinite(a).all()) and not torch.equal(a, b)
    assert rel_l2(a.double().cpu().numpy(), b.double().cpu().numpy()) < 1e-6
    assert abs(wa - wb) <= 1e-5 * abs(wb)
