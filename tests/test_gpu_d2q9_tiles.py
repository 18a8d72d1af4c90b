"""The multi-step D2Q9 kernels on every tile size (8, 16 and 32 nodes, chosen by
the grid) and with every option they take: a force field, a separate omega_p,
halfway and moving walls, link-wall distances, wall velocities link by link.
Fields must be bitwise those of one step per launch (variant GENERIC), and the
reverse sweep's mu bitwise that of separate reverse-step calls."""
import numpy as np
import pytest
import torch

import workloads as wl
from gpu_helpers import banner, need_gpu, to_dev

pytestmark = pytest.mark.gpu

GENERIC = 1
# on 256 compute units: tiles of 8, 8, 16 and 32; sides that leave remainders,
# and one smaller than a tile's region
SHAPES = [(1, 20, 12), (1, 70, 101), (1, 210, 203), (1, 401, 503)]
KINDS = ["plain", "walls force", "field", "omega_p", "omega_p walls", "q", "links", "q links force",
         "field walls"]


def _solver(L, shape, kind, variant):
    nz, ny, nx = shape
    rng = np.random.Generator(np.random.PCG64(121))
    kw = {}
    if any(k in kind for k in ("walls", "q ", "links")) or kind == "q":
        m = (rng.random(shape) < 0.04).astype(np.uint8) * rng.integers(1, 3, shape).astype(np.uint8)
        m[:, 0], m[:, -1] = 1, 2
        kw["mask"] = to_dev(m, torch.uint8)
        kw["wall_u"] = [list(r) for r in wl.wall_table((0.03, 0.01, 0.0))]
    if kind.startswith("q"):
        kw["qd"] = to_dev(rng.uniform(0.05, 1.0, (9,) + shape))
    if "force" in kind:
        kw["g"] = (1e-5, -2e-6)
    s = L.Solver(9, nx, ny, 1, 1.7, variant=variant,
                 omega_p=1.2 if "omega_p" in kind else None, **kw)
    if "field" in kind:
        s.set_force_field(to_dev(rng.uniform(-1e-5, 1e-5, (2,) + shape)))
    if "links" in kind:
        s.set_wall_velocity_links(to_dev(rng.uniform(-0.03, 0.03, (9, 2) + shape)))
    drho, u = wl.random_state(shape, 2, seed=123, du=0.03, drho=0.01)
    s.set_state(to_dev(drho), to_dev(u))
    return s


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("kind", KINDS)
def test_tiles_equal_single_steps(shape, kind):
    L = need_gpu()
    banner(f"d2q9 tiles {shape} {kind}")
    a, b = _solver(L, shape, kind, 0), _solver(L, shape, kind, GENERIC)
    for steps in (1, 8, 11):
        a.step(steps)
        b.step(steps)
        assert torch.equal(a.save_state(), b.save_state()), steps
        (ma, ea), (mb, eb) = a.diagnostics(), b.diagnostics()
        assert abs(ma - mb) <= 1e-12 * abs(mb) and abs(ea - eb) <= 1e-12 * abs(eb)
    st0, sb = a.save_state(), a.state_bytes
    out = torch.zeros(9 * sb, dtype=torch.uint8, device="cuda")
    L.lwacm_forward_states(a.ctx, st0, 0, 9, out)
    for k in range(9):
        a.step(1)
        assert torch.equal(out[k * sb:(k + 1) * sb], a.save_state())
    a.close()
    b.close()


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("kind", ["plain", "walls force"])
@pytest.mark.parametrize("t0", [0, 5])
def test_reverse_tiles_equal_separate_calls(shape, kind, t0):
    L = need_gpu()
    banner(f"d2q9 reverse tiles {shape} {kind} t0={t0}")
    s, n = _solver(L, shape, kind, 0), 11
    st = []
    for _ in range(n):
        st.append(s.save_state())
        s.step(1)
    g = torch.Generator(device="cuda")
    g.manual_seed(125)
    mu0 = torch.randn(shape + (3,), device="cuda", generator=g)
    mu, tmp = mu0.clone(), torch.empty_like(mu0)
    dw = torch.zeros(1, dtype=torch.float64, device="cuda")
    for j in range(n - 1, -1, -1):
        L.lwacm_adjoint_step(s.ctx, st[j], mu, tmp, dw, t0 + j == 0)
        mu, tmp = tmp, mu
    mu_s, dw_s = mu0.clone(), torch.zeros(1, dtype=torch.float64, device="cuda")
    L.lwacm_adjoint_sweep(s.ctx, torch.cat(st), t0, n, mu_s, torch.empty_like(mu0), dw_s)
    s.close()
    assert torch.equal(mu, mu_s)
    assert abs(float(dw) - float(dw_s)) <= 1e-12 * abs(float(dw)) + 1e-12
