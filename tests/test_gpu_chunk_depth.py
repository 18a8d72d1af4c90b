"""Chunk depths of the D3Q19 tile kernels are any number of planes: the depth
lwacm_init picks (unequal remainders of the rolled plane loop, a ragged last
chunk) against one chunk over all planes, bitwise in the fields for every
forward kernel, and the reverse kernels on such grids against the generic
reverse step (2e-6, the bound of the other comparisons of the two) and each
other (mu bitwise, dL/domega to the FP32 rounding of its partial sums)."""
import numpy as np
import pytest
import torch

import workloads as wl
from gpu_helpers import banner, need_gpu, rel_l2, to_dev

pytestmark = pytest.mark.gpu

MARCH, GENERIC = 2, 1


@pytest.mark.parametrize("nz", [23, 61, 100])  # depths 12, 9 and 9: every remainder with 8
@pytest.mark.parametrize("kind", ["single", "pairs", "fp16", "walls", "thermal"])
def test_chosen_depth_equals_one_chunk(nz, kind):
    L = need_gpu()
    shape = (nz, 16, 32)
    banner(f"chunk depth nz={nz} {kind}")
    drho, u = wl.random_state(shape, 3, seed=91, du=0.03, drho=0.01)
    mask = table = None
    if kind in ("walls", "thermal"):
        mask = np.zeros(shape, dtype=np.uint8)
        mask[0], mask[:, 0], mask[-1] = 1, 1, 2
        table = [list(r) for r in wl.wall_table((0.04, 0.01, 0.0))]
    out = []
    for planes in (0, 128):  # the chosen depth, then at most nz planes: one chunk
        s = L.Solver(19, 32, 16, nz, 1.7, storage=1 if kind == "fp16" else 0,
                     mask=None if mask is None else to_dev(mask, torch.uint8), wall_u=table,
                     variant=MARCH if kind == "single" else 0)
        if planes:
            L.lwacm_set_march_chunk(s.ctx, planes)
        s.set_state(to_dev(drho), to_dev(u))
        if kind == "thermal":
            s.set_thermal(1.4, to_dev(1.0 + drho), wall_T=(float("nan"), 0.9, 1.1))
        s.step(5)
        dr, uu = s.moments()
        out.append([dr, uu] + ([s.temperature()] if kind == "thermal" else []))
        m, e = s.diagnostics()
        assert abs(m - s.nx * s.ny * nz) < s.nx * s.ny * nz and e > 0.0
        s.close()
    for a, b in zip(*out):
        assert bool(torch.isfinite(a).all()) and torch.equal(a, b)


@pytest.mark.parametrize("nz", [8, 9, 10, 23, 61])
@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("final", [False, True])
def test_reverse_steps_of_any_depth(nz, walls, final):
    L = need_gpu()
    shape = (nz, 16, 32)
    banner(f"reverse chunk depth nz={nz} walls={walls} final={final}")
    drho, u = wl.random_state(shape, 3, seed=93, du=0.03, drho=0.01)
    mask = table = None
    if walls:
        mask = (np.random.Generator(np.random.PCG64(95)).random(shape) < 0.05).astype(np.uint8) * 2
        table = [list(r) for r in wl.wall_table((0.04, 0.01, 0.0))]
    s = L.Solver(19, 32, 16, nz, 1.6, mask=None if mask is None else to_dev(mask, torch.uint8),
                 wall_u=table)
    s.set_state(to_dev(drho), to_dev(u))
    st0 = s.save_state()
    s.step(1)
    st1 = s.save_state()
    rng = np.random.Generator(np.random.PCG64(97))
    mu0 = to_dev(rng.standard_normal(shape + (4,)) * 0.1)
    if walls:
        mu0[torch.as_tensor(mask != 0, device="cuda")] = 0.0

    def two():
        mid, out = torch.empty_like(mu0), torch.empty_like(mu0)
        dw = torch.zeros(1, dtype=torch.float64, device="cuda")
        L.lwacm_adjoint_step(s.ctx, st1, mu0, mid, dw, False)
        L.lwacm_adjoint_step(s.ctx, st0, mid, out, dw, final)
        return out, float(dw.item())

    a, wa = two()
    L.lwacm_set_variant(s.ctx, GENERIC)
    b, wb = two()
    L.lwacm_set_variant(s.ctx, 0)
    assert rel_l2(a.double().cpu().numpy(), b.double().cpu().numpy()) < 2e-6
    assert abs(wa - wb) <= 1e-5 * abs(wb) + 1e-6
    c = torch.empty_like(mu0)
    dw = torch.zeros(1, dtype=torch.float64, device="cuda")
    if L.lwacm_adjoint_step2(s.ctx, st1, st0, mu0, c, dw, final):
        assert torch.equal(a, c) and abs(wa - float(dw.item())) <= 1e-6 * abs(wa) + 1e-9
    else:
        assert walls
    s.close()
