"""D2Q9 tiles of 32 in more than one round, with walls or a separate omega_p: the
kernel with half the threads a workgroup, bitwise the one-step kernel (variant
GENERIC) in lwacm_step and lwacm_forward_states, eight steps and fewer."""
import numpy as np
import pytest
import torch

import workloads as wl
from gpu_helpers import banner, need_gpu, to_dev

pytestmark = pytest.mark.gpu

GENERIC = 1


@pytest.mark.parametrize("nx,ny", [(513, 545), (1031, 290)])  # 306 and 330 tiles
@pytest.mark.parametrize("kind", ["omega_p", "walls", "walls force", "walls omega_p", "walls field",
                                  "omega_p field"])
def test_paired_workgroups_equal_single_steps(nx, ny, kind):
    L = need_gpu()
    banner(f"pairs {nx}x{ny} {kind}")
    shape = (1, ny, nx)
    drho, u = wl.random_state(shape, 2, seed=109, du=0.03, drho=0.01)
    kw = dict(omega_p=1.2 if "omega_p" in kind else None, g=(1e-4, -2e-4) if "force" in kind else None)
    if "walls" in kind:
        m = (np.random.Generator(np.random.PCG64(109)).random(shape) < 0.01).astype(np.uint8)
        m[:, 0], m[:, -1] = 1, 2
        kw.update(mask=to_dev(m, torch.uint8), wall_u=[[0.0] * 3, [0.0] * 3, [0.04, 0.01, 0.0]])
    field = to_dev(1e-4 * np.random.Generator(np.random.PCG64(110)).standard_normal((2,) + shape))
    out = []
    for variant in (0, GENERIC):
        s = L.Solver(9, nx, ny, 1, 1.7, variant=variant, **kw)
        if "field" in kind:
            s.set_force_field(field)
        s.set_state(to_dev(drho), to_dev(u))
        st0 = s.save_state()
        slots = torch.empty(11 * s.state_bytes, dtype=torch.uint8, device="cuda")
        L.lwacm_forward_states(s.ctx, st0, 0, 11, slots)
        s.step(11)
        out.append(s.moments() + (s.save_state(), slots))
        s.close()
    for a, b in zip(*out):
        assert torch.equal(a, b)
    a = out[0]
    assert bool(torch.isfinite(a[0]).all() and torch.isfinite(a[1]).all())
    assert torch.equal(a[2], a[3][-a[2].numel():])
