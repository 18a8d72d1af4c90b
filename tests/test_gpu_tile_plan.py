"""Chunks of unequal depth in the D3Q19 tile kernels with walls: walls across x
cost more than walls across y, so lwacm_init cuts those tiles into shallower
chunks.  The fields are bitwise those of chunks of one depth
(lwacm_set_march_chunk), for every kernel that takes the list; the sums, FP32
per thread over another number of planes, agree to 2e-6 of the absolute values
summed.  Ragged sides (temperature) against the gather kernels, 1e-6."""
import numpy as np
import pytest
import torch

import workloads as wl
from gpu_helpers import banner, need_gpu, rel_l2, to_dev

pytestmark = pytest.mark.gpu

GENERIC, MARCH = 1, 2


def _solver(L, shape, **kw):
    nz, ny, nx = shape
    m = np.zeros(shape, dtype=np.uint8)
    m[:, :, 0], m[:, :, -1], m[:, 0], m[:, -1], m[-1] = 1, 1, 1, 1, 2
    m[nz // 3: nz // 2, ny // 3: ny // 2, : nx // 4] = 1  # a block in some of the tiles
    table = [list(r) for r in wl.wall_table((0.04, 0.01, 0.0))]
    s = L.Solver(19, nx, ny, nz, 1.7, mask=to_dev(m, torch.uint8), wall_u=table, **kw)
    drho, u = wl.random_state(shape, 3, seed=97, du=0.03, drho=0.01)
    s.set_state(to_dev(drho), to_dev(u))
    return s, drho


@pytest.mark.parametrize("shape", [(64, 64, 320), (101, 96, 160), (98, 80, 160)])
@pytest.mark.parametrize("kind", ["single", "pairs", "fp16", "force", "thermal"])
def test_unequal_chunks_equal_uniform_ones(shape, kind):
    L = need_gpu()
    banner(f"chunk list {shape} {kind}")
    out = []
    for planes in (0, 32):  # the chosen chunks, then 32 planes each
        s, drho = _solver(L, shape, storage=1 if kind == "fp16" else 0,
                          variant=MARCH if kind == "single" else 0,
                          g=(1e-4, -2e-4, 3e-4) if kind == "force" else None)
        if planes:
            L.lwacm_set_march_chunk(s.ctx, planes)
        if kind == "thermal":
            s.set_thermal(1.4, to_dev(1.0 + drho), wall_T=(float("nan"), 0.9, 1.1))
        s.step(5)
        dr, uu = s.moments()
        out.append([dr, uu] + ([s.temperature()] if kind == "thermal" else []) + [s.diagnostics()])
        s.close()
    for a, b in zip(out[0][:-1], out[1][:-1]):
        assert bool(torch.isfinite(a).all()) and torch.equal(a, b)
    (m0, e0), (m1, e1) = out[0][-1], out[1][-1]
    assert abs(m1 - m0) <= 2e-6 * float(out[0][0].double().abs().sum())
    assert abs(e1 - e0) <= 2e-6 * e0


@pytest.mark.parametrize("shape", [(75, 84, 250), (40, 33, 300)])
def test_unequal_chunks_on_ragged_sides(shape):
    L = need_gpu()
    banner(f"chunk list, ragged {shape}")
    out = []
    for variant in (0, GENERIC):
        s, drho = _solver(L, shape, variant=variant)
        s.set_thermal(1.4, to_dev(1.0 + drho), wall_T=(float("nan"), 0.9, 1.1))
        s.step(4)
        dr, uu = s.moments()
        out.append([t.double().cpu().numpy() for t in (dr, uu, s.temperature())])
        s.close()
    for x, y in zip(*out):
        assert rel_l2(x, y) < 1e-6
