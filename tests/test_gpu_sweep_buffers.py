"""lwacm_adjoint_sweep writes its arguments and nothing else of the caller's:
both state buffers of the context keep their bytes, on grids whose chunks fill
the chip and on grids whose dL/domega is summed in a pass of its own."""
import pytest
import torch

import workloads as wl
from gpu_helpers import banner, need_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q,shape,storage", [(19, (33, 16, 64), 0), (19, (96, 48, 32), 0),
                                             (19, (96, 48, 32), 1), (19, (100, 32, 32), 0),
                                             (19, (61, 65, 67), 0), (9, (1, 65, 130), 0)])
@pytest.mark.parametrize("t0", [0, 4])
def test_sweep_leaves_the_state_buffers(q, shape, storage, t0):
    L = need_gpu()
    nz, ny, nx = shape
    banner(f"sweep buffers q={q} {shape} storage={storage} t0={t0}")
    D = 2 if q == 9 else 3
    drho, u = wl.random_state(shape, D, seed=181, du=0.03, drho=0.01)
    s = L.Solver(q, nx, ny, nz, 1.6, storage=storage)
    s.set_state(to_dev(drho), to_dev(u))
    st = []
    for _ in range(3):
        st.append(s.save_state())
        s.step(1)
    before = s._a.clone(), s._b.clone()
    mu = torch.ones(nx * ny * nz * (D + 1), device="cuda")
    dw = torch.zeros(1, dtype=torch.float64, device="cuda")
    L.lwacm_adjoint_sweep(s.ctx, torch.cat(st), t0, 3, mu, torch.empty_like(mu), dw)
    assert torch.equal(s._a, before[0]) and torch.equal(s._b, before[1])
    s.close()
