"""What a solid node's fields hold (they are never updated, and nothing asks for
finite values there) must not reach the fluid: with NaN and infinities at the
solid nodes, the fluid's fields, the temperature, mass, energy and mu are
bitwise those of the same run with zeros there, on every kernel that takes walls."""
import numpy as np
import pytest
import torch

import workloads as wl
from gpu_helpers import banner, need_gpu, to_dev

pytestmark = pytest.mark.gpu

GENERIC, MARCH = 1, 2
RAGGED = [(9, 17, 33), (20, 35, 70)]
CASES = ([(19, s, k) for s in RAGGED for k in ("thermal", "walls", "fp16", "force", "q", "links")] +
         [(19, (20, 32, 64), k) for k in ("thermal", "single", "walls", "fp16", "force", "q")] +
         [(19, (5, 16, 32), k) for k in ("walls", "fp16")] +
         [(9, (1, 40, 70), k) for k in ("walls", "force", "omega_p", "q", "links")] +
         [(9, (1, 300, 257), "walls"), (9, (1, 545, 513), "walls")])


def _geometry(q, shape):
    rng = np.random.Generator(np.random.PCG64(151))
    m = (rng.random(shape) < 0.03).astype(np.uint8)
    m[:, :, 0], m[:, -1] = 1, 2
    drho, u = wl.random_state(shape, 2 if q == 9 else 3, seed=153, du=0.03, drho=0.01)
    return m, drho, u


def _garbage(a, m, rng):
    """a with NaN and both infinities at the solid nodes."""
    a = np.array(a, dtype=np.float32)
    a[..., m != 0] = rng.choice([np.nan, np.inf, -np.inf], a[..., m != 0].shape)
    return a


def _solver(L, q, shape, kind, m, drho, u, T=None):
    nz, ny, nx = shape
    rng = np.random.Generator(np.random.PCG64(155))
    links = (q, 2 if q == 9 else 3) + shape
    s = L.Solver(q, nx, ny, nz, 1.7, storage=1 if kind == "fp16" else 0, mask=to_dev(m, torch.uint8),
                 wall_u=[[0.0] * 3, [0.0] * 3, [0.04, 0.01, 0.0]],
                 variant=MARCH if kind == "single" else 0,
                 g=(1e-4, -2e-4, 3e-4)[: 2 if q == 9 else 3] if kind == "force" else None,
                 omega_p=1.2 if kind == "omega_p" else None,
                 qd=to_dev(rng.uniform(0.05, 1.0, (q,) + shape)) if kind == "q" else None)
    if kind == "links":
        s.set_wall_velocity_links(to_dev(rng.uniform(-0.03, 0.03, links)))
    s.set_state(to_dev(drho), to_dev(u))
    if T is not None:
        s.set_thermal(1.4, to_dev(T), wall_T=(float("nan"), 0.9, float("nan")))
    return s


@pytest.mark.parametrize("q,shape,kind", CASES)
def test_values_at_solid_nodes_stay_there(q, shape, kind):
    L = need_gpu()
    banner(f"solid values q={q} {shape} {kind}")
    m, drho, u = _geometry(q, shape)
    rng = np.random.Generator(np.random.PCG64(157))
    out = []
    for garbage in (False, True):
        put = (lambda a: _garbage(a, m, rng)) if garbage else (lambda a: np.where(m != 0, 0.0, a))
        s = _solver(L, q, shape, kind, m, put(drho), put(u),
                    put(1.0 + drho) if kind == "thermal" else None)
        got = []
        for steps in (1, 4, 9):
            s.step(steps)
            got += list(s.moments()) + ([s.temperature()] if kind == "thermal" else [])
        out.append(([t[..., to_dev(m, torch.uint8) == 0] for t in got], s.diagnostics()))
        s.close()
    for a, b in zip(out[0][0], out[1][0]):
        assert bool(torch.isfinite(a).all()) and torch.equal(a, b)
    assert out[0][1] == out[1][1]


@pytest.mark.parametrize("q,shape", [(19, (20, 32, 64)), (19, (5, 16, 32)), (19, (9, 17, 33)),
                                     (9, (1, 40, 70))])
@pytest.mark.parametrize("t0", [0, 5])
def test_reverse_steps_ignore_states_of_solid_nodes(q, shape, t0):
    L = need_gpu()
    banner(f"reverse, solid values q={q} {shape} t0={t0}")
    m, drho, u = _geometry(q, shape)
    rng = np.random.Generator(np.random.PCG64(159))
    D, n = (2 if q == 9 else 3), int(np.prod(shape))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(161)
    lam = torch.randn((D + 1,) + shape, device="cuda", generator=gen)
    out = []
    for put in (lambda a: np.where(m != 0, 0.0, a), lambda a: _garbage(a, m, rng)):
        s = _solver(L, q, shape, "walls", m, put(drho), put(u))
        st = []
        for _ in range(3):
            st.append(s.save_state())
            s.step(1)
        mu, tmp = torch.empty(n * (D + 1), device="cuda"), torch.empty(n * (D + 1), device="cuda")
        dw = torch.zeros(1, dtype=torch.float64, device="cuda")
        L.lwacm_adjoint_seed(s.ctx, s.save_state(), lam, mu)
        L.lwacm_adjoint_sweep(s.ctx, torch.cat(st), t0, 3, mu, tmp, dw)
        out.append((mu, float(dw)))
        s.close()
    assert bool(torch.isfinite(out[0][0]).all()) and torch.equal(out[0][0], out[1][0])
    assert out[0][1] == out[1][1]
