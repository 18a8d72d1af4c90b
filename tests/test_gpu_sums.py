"""Mass and energy of a step against FP64 sums of the fields it leaves, as
lwacm_moments forms them.  With a temperature on sides that are no multiples of
the tile every kernel adds node by node in FP64, so the two agree to its
rounding: 1e-12 of the absolute values summed.  Without one the tile kernels add a
thread's planes in FP32, but no more of them in one sum than the depths 32, 64
and 128 gave a thread: 32 at 256 x 256 x 192, where the chunks are 96 deep."""
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


def _chain_errors(v, n):
    """Relative errors of the FP32 sums of 1 .. n equal terms v."""
    acc, out = np.float32(0.0), []
    for k in range(1, n + 1):
        acc = np.float32(v + np.float64(acc))
        out.append(abs(float(acc) - k * v) / (k * v))
    return np.array(out)


@pytest.mark.parametrize("kind", ["pairs", "single", "fp16", "walls"])
def test_fp32_sums_stay_short_in_deep_chunks(kind):
    """A uniform flow keeps its velocity and gives every node the same energy, chosen
    so that 96 of them in one FP32 sum lose more than five times what any sum of at
    most 32 does: the tolerance is that maximum."""
    L = need_gpu()
    banner(f"deep chunks {kind}")
    nx, ny, nz = 256, 256, 192
    ux = 2005.0 / 65536.0  # 11 bits: exact in FP16 storage too
    err = _chain_errors(ux * ux, 96)
    assert err[95] > 5.0 * err[:32].max()
    kw = {}
    if kind == "walls":  # the masked kernels, with no solid node
        kw = dict(mask=torch.zeros((nz, ny, nx), dtype=torch.uint8, device="cuda"))
    s = L.Solver(19, nx, ny, nz, 1.7, storage=1 if kind == "fp16" else 0,
                 variant=2 if kind == "single" else 0, **kw)
    u = torch.zeros((3, nz, ny, nx), device="cuda")
    u[0] = ux
    s.set_state(torch.zeros((nz, ny, nx), device="cuda"), u)
    hist = torch.zeros(8, dtype=torch.float64, device="cuda")
    L.lwacm_set_diag_history(s.ctx, hist)
    s.step(2)
    dr, uu = s.moments()
    assert bool((uu[0] == ux).all()) and not bool(uu[1:].any())
    s.close()
    exact = 0.5 * nx * ny * nz * ux * ux
    for step in (1, 2):
        assert abs(float(hist[2 * step + 1]) - exact) <= 1.001 * err[:32].max() * exact


def test_pairs_and_single_steps_split_their_sums_alike():
    L = need_gpu()
    nx, ny, nz = 256, 160, 200  # chunks of 67 planes, sums of 32
    banner("deep chunks, pairs and single steps")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(195)
    u = 0.02 * torch.randn((3, nz, ny, nx), device="cuda", generator=gen)
    out = []
    for variant in (0, 2):
        s = L.Solver(19, nx, ny, nz, 1.7, variant=variant)
        hist = torch.zeros(16, dtype=torch.float64, device="cuda")
        L.lwacm_set_diag_history(s.ctx, hist)
        s.set_state(0.1 * u[0], u)
        s.step(5)
        s.diagnostics()
        out.append((hist, s.save_state()))
        s.close()
    assert torch.equal(out[0][1], out[1][1]) and torch.equal(out[0][0], out[1][0])
