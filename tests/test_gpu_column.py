"""D3Q19 grids that the tile kernels do not take run the column-marching gather
kernels: fields (solid nodes included), FP16 bits, states of a segment and mu
must be bitwise those of the one-thread-per-node kernels (variant GENERIC), mass,
energy and dL/domega equal to FP64 rounding, on sides around multiples of the
tile, sides of one node, few planes, and with every option the kernels take.  (Without
walls the column kernels start at 10^5 nodes, FP16 at 2.5 10^5.)"""
import numpy as np
import pytest
import torch

import workloads as wl
from gpu_helpers import banner, need_gpu, to_dev

pytestmark = pytest.mark.gpu

GENERIC = 1
SHAPES = [(1, 1, 1), (2, 3, 5), (9, 17, 33), (7, 70, 40), (33, 15, 64), (2, 401, 399),
          (61, 65, 67), (1025, 16, 16)]
KINDS = ["plain", "fp16", "fp16 nearest", "force", "field", "walls", "walls field", "walls fp16",
         "q force", "q links", "links fp16"]


def _solver(L, shape, kind, variant):
    nz, ny, nx = shape
    rng = np.random.Generator(np.random.PCG64(131))
    kw = {}
    if any(k in kind for k in ("walls", "q ", "links")):
        m = (rng.random(shape) < 0.05).astype(np.uint8) * rng.integers(1, 3, shape).astype(np.uint8)
        m[:, -1] = 2
        kw["mask"] = to_dev(m, torch.uint8)
        kw["wall_u"] = [list(r) for r in wl.wall_table((0.03, 0.01, -0.02))]
    if "q " in kind:
        kw["qd"] = to_dev(rng.uniform(0.05, 1.0, (19,) + shape))
    if "force" in kind:
        kw["g"] = (1e-5, -2e-6, 3e-6)
    s = L.Solver(19, nx, ny, nz, 1.7, storage=1 if "fp16" in kind else 0, variant=variant,
                 fp16_rounding=(0, 0) if "nearest" in kind else None, **kw)
    if "field" in kind:
        s.set_force_field(to_dev(rng.uniform(-1e-5, 1e-5, (3,) + shape)))
    if "links" in kind:
        s.set_wall_velocity_links(to_dev(rng.uniform(-0.03, 0.03, (19, 3) + shape)))
    drho, u = wl.random_state(shape, 3, seed=133, du=0.03, drho=0.01)
    s.set_state(to_dev(drho), to_dev(u))
    return s


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("kind", KINDS)
def test_columns_equal_the_generic_kernel(shape, kind):
    L = need_gpu()
    banner(f"columns {shape} {kind}")
    a, b = _solver(L, shape, kind, 0), _solver(L, shape, kind, GENERIC)
    for steps in (1, 4):
        a.step(steps)
        b.step(steps)
        assert torch.equal(a.save_state(), b.save_state()), steps
        (ma, ea), (mb, eb) = a.diagnostics(), b.diagnostics()
        assert abs(ma - mb) <= 1e-12 * abs(mb) and abs(ea - eb) <= 1e-12 * abs(eb) + 1e-30
    st0, sb = a.save_state(), a.state_bytes
    out = torch.zeros(2 * sb, dtype=torch.uint8, device="cuda")
    L.lwacm_forward_states(a.ctx, st0, a.step_count, 2, out)
    for k in range(2):
        b.step(1)
        assert torch.equal(out[k * sb:(k + 1) * sb], b.save_state())
    a.close()
    b.close()


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("kind", ["plain", "fp16", "force"])
@pytest.mark.parametrize("t0", [0, 5])
def test_reverse_columns_equal_the_generic_kernel(shape, kind, t0):
    L = need_gpu()
    banner(f"reverse columns {shape} {kind} t0={t0}")
    s, n = _solver(L, shape, kind, 0), 3
    st = []
    for _ in range(n):
        st.append(s.save_state())
        s.step(1)
    g = torch.Generator(device="cuda")
    g.manual_seed(135)
    mu0 = torch.randn(shape + (4,), device="cuda", generator=g)

    def separate():
        mu, tmp = mu0.clone(), torch.empty_like(mu0)
        dw = torch.zeros(1, dtype=torch.float64, device="cuda")
        for j in range(n - 1, -1, -1):
            L.lwacm_adjoint_step(s.ctx, st[j], mu, tmp, dw, t0 + j == 0)
            mu, tmp = tmp, mu
        return mu, float(dw)

    a, wa = separate()
    mu_s, dw = mu0.clone(), torch.zeros(1, dtype=torch.float64, device="cuda")
    L.lwacm_adjoint_sweep(s.ctx, torch.cat(st), t0, n, mu_s, torch.empty_like(mu0), dw)
    assert torch.equal(a, mu_s) and wa == float(dw)
    L.lwacm_set_variant(s.ctx, GENERIC)
    b, wb = separate()
    s.close()
    assert torch.equal(a, b) and abs(wa - wb) <= 1e-12 * abs(wb) + 1e-12
