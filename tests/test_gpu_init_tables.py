"""What lwacm_init and lwacm_set_thermal allocate on masked D3Q19 grids whose sides
are no multiples of the tile: lwacm_init the node classes and the wall list of
the column kernels (1 byte a node and 4 a listed node) but none of the tile
kernels' tables, which only a temperature needs (12 bytes a node more, 28 with
moving walls)."""
import pytest
import torch

from gpu_helpers import banner, need_gpu

pytestmark = pytest.mark.gpu

SLACK = 16 << 20  # partials, lists, allocation granules


def _free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


@pytest.mark.parametrize("moving", [False, True])
def test_tables_of_ragged_masked_grids(moving):
    L = need_gpu()
    nz, ny, nx = 301, 303, 299
    banner(f"tables {(nz, ny, nx)} moving={moving}")
    n = nx * ny * nz
    mask = torch.zeros((nz, ny, nx), dtype=torch.uint8, device="cuda")
    mask[0], mask[-1] = 1, 2
    a = torch.empty(16 * n, dtype=torch.uint8, device="cuda")
    b = torch.empty_like(a)
    T = torch.ones((2, n), device="cuda")
    wall_u = [[0.0] * 3, [0.0] * 3, [0.05 if moving else 0.0, 0.0, 0.0]]
    before = _free()
    ctx = L.lwacm_init(19, nx, ny, nz, 1.7, 0, a, b, mask, wall_u, None,
                       L._stream_handle(a.device))
    after = _free()
    assert before - after <= n + 4 * 2 * nx * ny + SLACK
    L.lwacm_set_thermal(ctx, 1.4, T[0], T[1], (float("nan"), 0.9, 1.1))
    assert after - _free() <= (28 if moving else 12) * n + SLACK
    L.lwacm_destroy(ctx)
    assert before - _free() <= SLACK
