"""FP16 storage rounded to nearest: a step of the tile kernel is the FP32 step of the
dequantised state, rounded to FP32 and then to FP16 -- bit for bit, on plain
problems and with walls (halfway, interpolated), where velocities stay in
units of the storage scale throughout, and with a force and omega_p, where they
do not."""
import numpy as np
import pytest
import torch

import workloads as wl
from gpu_helpers import banner, need_gpu, to_dev

pytestmark = pytest.mark.gpu

MARCH = 2


@pytest.mark.parametrize("shape", [(5, 16, 32), (20, 32, 64), (40, 48, 96)])
@pytest.mark.parametrize("kind", ["plain", "walls", "q", "force", "omega_p"])
@pytest.mark.parametrize("scales", [(14, 14), (12, 16)])
def test_a_step_rounds_to_fp32_then_to_fp16(shape, kind, scales):
    L = need_gpu()
    nz, ny, nx = shape
    if nz < 8 and kind in ("force", "omega_p"):
        pytest.skip("not on the tile kernel")
    banner(f"FP16 nearest {shape} {kind} {scales}")
    rng = np.random.Generator(np.random.PCG64(241))
    kw = {}
    if kind in ("walls", "q"):
        m = (rng.random(shape) < 0.04).astype(np.uint8)
        m[:, :, 0], m[:, -1] = 1, 2
        # at rest: set_state, called before every FP32 step, sets the density of
        # the moving-wall term anew
        kw = dict(mask=to_dev(m, torch.uint8), wall_u=[[0.0] * 3] * 3)
    if kind == "q":
        kw["qd"] = to_dev(rng.uniform(0.05, 1.0, (19,) + shape))
    if kind == "force":
        kw["g"] = (1e-5, -2e-6, 3e-6)
    if kind == "omega_p":
        kw["omega_p"] = 1.3
    drho, u = wl.random_state(shape, 3, seed=243, du=0.03, drho=0.01)
    h = L.Solver(19, nx, ny, nz, 1.7, storage=1, variant=MARCH, fp16_scales=scales,
                 fp16_rounding=(0, 0), **kw)
    h.set_state(to_dev(drho), to_dev(u))
    s = L.Solver(19, nx, ny, nz, 1.7, variant=MARCH, **kw)
    for step in range(3):
        dr, uu = h.moments()  # exact in FP32
        s.set_state(dr, uu)
        s.step(1)
        h.step(1)
        f = s.save_state().view(torch.float32).view(-1, 4).clone()
        f[:, 0] *= 2.0 ** scales[0]
        f[:, 1:] *= 2.0 ** scales[1]
        got = h.save_state().view(torch.float16).view(-1, 4)
        assert torch.equal(got, f.to(torch.float16)), (step, int((got != f.to(torch.float16)).sum()))
    h.close()
    s.close()
