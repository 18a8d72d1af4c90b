"""A mask may start at any byte: lwacm_init counts its fluid nodes and finds ids out
of range wherever they lie (before the first 16-byte boundary, in whole words,
after the last), and an edit of any single node is seen by the next step."""
import pytest
import torch

import workloads as wl
from gpu_helpers import banner, need_gpu, to_dev

pytestmark = pytest.mark.gpu

SHAPE = (7, 18, 35)  # 4410 nodes: 275 words of 16 bytes and 10 bytes more


def _mask(offset):
    n = SHAPE[0] * SHAPE[1] * SHAPE[2]
    base = torch.zeros(n + 32, dtype=torch.uint8, device="cuda")
    assert base.data_ptr() % 16 == 0
    return base[offset: offset + n].view(SHAPE)


@pytest.mark.parametrize("offset", [0, 1, 7, 15])
@pytest.mark.parametrize("q", [9, 19])
def test_scan_of_an_unaligned_mask(offset, q):
    L = need_gpu()
    banner(f"mask at byte {offset} q={q}")
    nz, ny, nx = SHAPE if q == 19 else (1, SHAPE[0] * SHAPE[1], SHAPE[2])
    n = nx * ny * nz
    for node in (0, 14, 15, 16, n // 2, n - 11, n - 1):
        m = _mask(offset).view(nz, ny, nx)
        m.view(-1)[node] = 1
        s = L.Solver(q, nx, ny, nz, 1.7, mask=m)
        assert s.mask.data_ptr() == m.data_ptr()
        u = torch.zeros((2 if q == 9 else 3, nz, ny, nx), device="cuda")
        s.set_state(u[0], u)
        s.step(1)
        assert s.diagnostics() == (float(n - 1), 0.0)
        s.close()
        m.view(-1)[node] = 3
        with pytest.raises(L.LWACMError) as e:
            L.Solver(q, nx, ny, nz, 1.7, mask=m)
        assert e.value.code == L.LWACM_EINVAL


@pytest.mark.parametrize("offset", [0, 1, 15])
def test_edits_of_single_nodes_are_seen(offset):
    L = need_gpu()
    banner(f"edits of single nodes, mask at byte {offset}")
    nz, ny, nx = SHAPE
    n = nx * ny * nz
    drho, u = wl.random_state(SHAPE, 3, seed=231, du=0.03, drho=0.01)
    for node in (0, 15, 16, n // 2, n - 1):
        out = []
        for variant in (0, 1):
            s = L.Solver(19, nx, ny, nz, 1.7, mask=_mask(offset), variant=variant)
            s.set_state(to_dev(drho), to_dev(u))
            s.mask.view(-1)[node] = 1
            s.step(2)
            out.append(s.save_state())
            s.close()
        assert torch.equal(*out), node
