"""Grids that the tile kernels do not take follow the mask and the link
distances as they are at each call: edited in place between calls, on D3Q19
grids with sides that are no multiples of the tile, the next steps are bitwise
those of the one-thread-per-node kernels (variant GENERIC, which read the mask at
every node and step); with a temperature, whose step runs in the flow's tile
kernel there, all fields within 1e-6."""
import numpy as np
import pytest
import torch

import workloads as wl
from gpu_helpers import banner, need_gpu, rel_l2, to_dev

pytestmark = pytest.mark.gpu

GENERIC = 1
SHAPES = [(9, 17, 33), (33, 15, 64), (61, 65, 67)]


def _mask(shape, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    m = (rng.random(shape) < 0.04).astype(np.uint8) * rng.integers(1, 3, shape).astype(np.uint8)
    m[:, seed % 5] = 1 + seed % 2
    return to_dev(m, torch.uint8)


def _solver(L, shape, kind, variant):
    nz, ny, nx = shape
    rng = np.random.Generator(np.random.PCG64(163))
    s = L.Solver(19, nx, ny, nz, 1.7, storage=1 if kind == "fp16" else 0, variant=variant,
                 mask=_mask(shape, 171),  # a tensor of the solver's own
                 wall_u=[list(r) for r in wl.wall_table((0.03, 0.01, -0.02))],
                 g=(1e-5, -2e-6, 3e-6) if kind == "force" else None,
                 qd=to_dev(rng.uniform(0.05, 1.0, (19,) + shape)) if kind == "q" else None)
    if kind == "links":
        s.set_wall_velocity_links(to_dev(rng.uniform(-0.03, 0.03, (19, 3) + shape)))
    drho, u = wl.random_state(shape, 3, seed=165, du=0.03, drho=0.01)
    s.set_state(to_dev(drho), to_dev(u))
    return s, drho


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("kind", ["walls", "fp16", "force", "q", "links"])
def test_steps_follow_the_edited_mask(shape, kind):
    L = need_gpu()
    banner(f"mask edits {shape} {kind}")
    (a, _), (b, _) = _solver(L, shape, kind, 0), _solver(L, shape, kind, GENERIC)
    # walls appear, vanish, change id, come back as they were
    for seed, steps in ((171, 2), (172, 1), (173, 3), (171, 2), (174, 1)):
        for s in (a, b):
            s.mask.copy_(_mask(shape, seed))
            if kind == "q":
                s.qd.mul_(0.9)
            s.step(steps)
        assert torch.equal(a.save_state(), b.save_state()), seed
        (ma, ea), (mb, eb) = a.diagnostics(), b.diagnostics()
        assert abs(ma - mb) <= 1e-12 * abs(mb) and abs(ea - eb) <= 1e-12 * abs(eb)
    st0, sb = a.save_state(), a.state_bytes
    out = torch.zeros(2 * sb, dtype=torch.uint8, device="cuda")
    for s in (a, b):
        s.mask.copy_(_mask(shape, 175))
    L.lwacm_forward_states(a.ctx, st0, a.step_count, 2, out)
    for k in range(2):
        b.step(1)
        assert torch.equal(out[k * sb:(k + 1) * sb], b.save_state())
    a.close()
    b.close()


def test_wall_force_lists_the_nodes_at_its_first_call():
    L = need_gpu()
    shape = (20, 35, 70)
    banner(f"mask edits, wall force {shape}")
    out = []
    for variant in (0, GENERIC):
        s, _ = _solver(L, shape, "walls", variant)
        s.step(1)
        s.mask.copy_((_mask(shape, 176) != 0).to(torch.uint8))
        out.append(s.wall_force(1, (3.0, 4.0, 5.0)))
        s.close()
    # the same list and the same sums
    s, _ = _solver(L, shape, "walls", 0)
    s.step(1)
    st = s.save_state()
    nz, ny, nx = shape
    r = L.Solver(19, nx, ny, nz, 1.7, mask=(_mask(shape, 176) != 0).to(torch.uint8))
    r.load_state(st)
    out.append(r.wall_force(1, (3.0, 4.0, 5.0)))
    s.close()
    r.close()
    assert out[0] == out[1] == out[2]


@pytest.mark.parametrize("shape", [(9, 17, 33), (61, 65, 67)])
def test_temperature_follows_the_edited_mask(shape):
    L = need_gpu()
    banner(f"mask edits, temperature {shape}")
    out = []
    for variant in (0, GENERIC):
        s, drho = _solver(L, shape, "walls", variant)
        s.set_thermal(1.4, to_dev(1.0 + drho), wall_T=(float("nan"), 0.9, 1.1))
        got = []
        for seed, steps in ((171, 1), (172, 1), (173, 2), (171, 1)):
            s.mask.copy_(_mask(shape, seed))
            s.step(steps)
            solid = (s.mask != 0).reshape(shape)
            fields = list(s.moments()) + [s.temperature()]
            got.append(([f[..., ~solid].double().cpu().numpy() for f in fields],
                        [f[..., solid] for f in fields]))
        out.append(got)
        s.close()
    for k, ((fa, sa), (fb, sb)) in enumerate(zip(*out)):
        for x, y in zip(fa, fb):
            assert rel_l2(x, y) < 1e-6, k
        for x, y in zip(sa, sb):
            # a node that turned solid keeps what the fluid had there
            assert rel_l2(x.double().cpu().numpy(), y.double().cpu().numpy()) < 1e-6, k
