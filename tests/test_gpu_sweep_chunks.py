"""Reverse sweeps on grids that the reverse tile kernels' deep chunks leave
partly empty run shallower chunks and sum dL/domega in a pass of its own: mu
and dL/domega must be bitwise those of separate reverse-step calls, with
odd counts, FP16 states, chunks of every remainder
and a grid whose last chunk is ragged."""
import numpy as np
import pytest
import torch

import workloads as wl
from gpu_helpers import banner, need_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,steps,storage,t0", [
    ((8, 16, 32), 4, 0, 0), ((33, 16, 64), 5, 0, 0), ((61, 32, 64), 6, 1, 0),
    ((96, 48, 32), 7, 0, 3), ((96, 48, 32), 7, 1, 0), ((100, 32, 32), 3, 0, 0), ((130, 16, 32), 1, 0, 2),
    ((192, 192, 192), 13, 0, 0)])  # the largest of them
def test_sweep_equals_separate_calls(shape, steps, storage, t0):
    L = need_gpu()
    nz, ny, nx = shape
    banner(f"sweep chunks {shape} steps={steps} storage={storage}")
    drho, u = wl.random_state(shape, 3, seed=111, du=0.03, drho=0.01)
    s = L.Solver(19, nx, ny, nz, 1.6, storage=storage)
    s.set_state(to_dev(drho), to_dev(u))
    st = []
    for _ in range(steps):
        st.append(s.save_state())
        s.step(1)
    g = torch.Generator(device="cuda")
    g.manual_seed(113)
    mu0 = 0.1 * torch.randn(shape + (4,), device="cuda", generator=g)
    mu, tmp = mu0.clone(), torch.empty_like(mu0)
    dw = torch.full((1,), 0.25, dtype=torch.float64, device="cuda")
    j = steps - 1
    while j >= 0:
        if j >= 1 and L.lwacm_adjoint_step2(s.ctx, st[j], st[j - 1], mu, tmp, dw, t0 + j == 1):
            j -= 2
        else:
            L.lwacm_adjoint_step(s.ctx, st[j], mu, tmp, dw, t0 + j == 0)
            j -= 1
        mu, tmp = tmp, mu
    mu_s, dw_s = mu0.clone(), torch.full((1,), 0.25, dtype=torch.float64, device="cuda")
    L.lwacm_adjoint_sweep(s.ctx, torch.cat(st), t0, steps, mu_s, torch.empty_like(mu0), dw_s)
    s.close()
    assert bool(torch.isfinite(mu).all()) and torch.equal(mu, mu_s)
    assert float(dw.item()) == float(dw_s.item())
