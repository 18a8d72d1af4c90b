"""lwacm_step_static takes the kernels of a context's lwacm_step at every size: state,
mass and energy bitwise equal on grids of the column and the strip kernels, with
launches of fewer steps after the strips, and at sizes whose kernels would need
more blocks than the fixed scratch holds (8192): D2Q9 of more than 8192 tiles
and D3Q19 of as many column workgroups."""
import pytest
import torch

from gpu_helpers import banner, need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q,shape,nsteps", [
    (19, (61, 65, 67), 3), (19, (130, 75, 101), 4),  # columns
    (9, (1, 1003, 1501), 19), (9, (1, 724, 724), 8),  # strips
    (9, (1, 130, 257), 11), (9, (1, 545, 513), 9),  # tiles
    (9, (1, 2304, 4096), 11), (9, (1, 2304, 4096), 16), (9, (1, 3000, 3001), 3),
    (19, (410, 407, 409), 2)])
def test_static_steps_take_the_context_kernels(q, shape, nsteps):
    L = need_gpu()
    nz, ny, nx = shape
    banner(f"static kernels q={q} {shape} x {nsteps}")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(201)
    D = 2 if q == 9 else 3
    u = 0.02 * torch.randn((D,) + shape, device="cuda", generator=gen)
    s = L.Solver(q, nx, ny, nz, 1.7)
    s.set_state(0.1 * u[0], u)
    a = s.save_state().view(torch.float32)
    s.step(nsteps)
    ref, (mass, energy) = s.save_state(), s.diagnostics()
    s.close()
    diag = torch.zeros(2, dtype=torch.float64, device="cuda")
    out = L.lwacm_step_static(q, nx, ny, nz, 1.7, a, torch.empty_like(a), nsteps, diag)
    assert torch.equal(out.view(torch.uint8), ref)
    assert float(nx * ny * nz) + float(diag[0]) == mass and float(diag[1]) == energy
