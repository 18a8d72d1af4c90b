"""Which kernel a problem runs on, by the names in a trace of one call, where the
choice follows sizes: the column kernels against one thread per node, strips
against tiles with and without omega_p, tiles of half the threads, the reverse
tile kernel on flat grids.  For a device of 256 CUs."""
import pytest
import torch
from torch.profiler import ProfilerActivity, profile

from gpu_helpers import banner, need_gpu

pytestmark = pytest.mark.gpu

FP16, WALLS, FORCE, FIELD, SPLIT, HEAT = "fp16", "walls", "force", "field", "omega_p", "heat"
COLUMN, GENERIC, TILE, TILE2 = "k_fwd_column", "k_fwd_generic", "k_fwd_march_rolled", "k_fwd_march2"
MULTI, STRIP = "k_fwd_d2q9_multi", "k_fwd_d2q9_strip"
FORWARD = [
    (19, (49, 49, 49), (), COLUMN), (19, (45, 45, 45), (), GENERIC),
    (19, (57, 57, 57), (FP16,), GENERIC), (19, (76, 76, 76), (FP16,), COLUMN),
    (19, (4, 1, 90001), (), COLUMN), (19, (4, 90001, 1), (FORCE,), COLUMN),
    (19, (4, 1, 90001), (FIELD, FP16), COLUMN), (19, (2, 300, 301), (), COLUMN),
    (19, (1, 400, 401), (), GENERIC), (19, (20000, 3, 3), (), GENERIC),
    (19, (4000, 8, 9), (FORCE,), GENERIC), (19, (3000, 17, 17), (FP16,), GENERIC),
    (19, (9, 9, 9), (WALLS,), COLUMN), (19, (1, 1, 300), (WALLS, FP16), COLUMN),
    (19, (1, 400, 401), (WALLS, FORCE), COLUMN), (19, (9001, 3, 3), (WALLS,), GENERIC),
    (19, (61, 65, 67), (WALLS, SPLIT), GENERIC), (19, (61, 65, 67), (WALLS, HEAT), TILE),
    (19, (57, 57, 57), (HEAT,), TILE), (19, (32, 33, 34), (HEAT,), GENERIC),
    (19, (64, 64, 64), (), TILE2), (19, (64, 64, 64), (FP16,), TILE),
    (9, (1, 961, 1009), (SPLIT,), MULTI), (9, (1, 1003, 1501), (SPLIT,), STRIP),
    (9, (1, 961, 1009), (), STRIP), (9, (1, 512, 512), (), MULTI),
]
REVERSE = [
    ((57, 57, 57), (), "k_adj_column"), ((45, 45, 45), (), "k_adj_generic"),
    ((76, 76, 76), (FP16,), "k_adj_column"), ((57, 57, 57), (FP16,), "k_adj_generic"),
    ((3, 300, 301), (), "k_adj_generic"), ((20000, 3, 3), (), "k_adj_generic"),
    ((1, 16, 32), (), "k_adj_march"), ((7, 16, 32), (WALLS,), "k_adj_march"),
    ((40, 16, 32), (), "k_adj_march"), ((57, 57, 57), (WALLS,), "k_adj_generic"),
]


def _solver(L, q, shape, kind):
    nz, ny, nx = shape
    kw = {}
    if WALLS in kind:
        m = torch.zeros(shape, dtype=torch.uint8, device="cuda")
        m[:, :, 0] = 1
        kw = dict(mask=m)
    s = L.Solver(q, nx, ny, nz, 1.7, storage=1 if FP16 in kind else 0,
                 g=(1e-6,) * (2 if q == 9 else 3) if FORCE in kind else None,
                 omega_p=1.2 if SPLIT in kind else None, **kw)
    u = torch.zeros((2 if q == 9 else 3,) + shape, device="cuda")
    s.set_state(u[0], u)
    if FIELD in kind:
        s.set_force_field(u)
    if HEAT in kind:
        s.set_thermal(1.4, 1.0 + u[0])
    return s


def _kernels(call):
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as trace:
        call()
        torch.cuda.synchronize()
    names = " ".join(e.key for e in trace.key_averages() if "lwacm" in e.key)
    if not names:
        pytest.skip("no trace of kernels here")
    return names


@pytest.mark.parametrize("q,shape,kind,kernel", FORWARD)
def test_forward_routes(q, shape, kind, kernel):
    L = need_gpu()
    banner(f"route q={q} {shape} {kind}")
    s = _solver(L, q, shape, kind)
    s.step(8)
    names = _kernels(lambda: s.step(8))
    s.close()
    assert kernel + "<" in names, names


@pytest.mark.parametrize("shape,kind,kernel", REVERSE)
def test_reverse_routes(shape, kind, kernel):
    L = need_gpu()
    banner(f"reverse route {shape} {kind}")
    s = _solver(L, 19, shape, kind)
    mu = torch.zeros(shape + (4,), device="cuda")
    out, dw = torch.empty_like(mu), torch.zeros(1, dtype=torch.float64, device="cuda")
    st = s.save_state()
    names = _kernels(lambda: L.lwacm_adjoint_step(s.ctx, st, mu, out, dw, False))
    s.close()
    assert kernel + "<" in names, names


@pytest.mark.parametrize("kind,pair", [((WALLS,), True), ((SPLIT,), True), ((FORCE, SPLIT), True),
                                       ((WALLS, FORCE), True), ((WALLS, SPLIT), True),
                                       ((FIELD, SPLIT), False), ((WALLS, FIELD), False),
                                       ((WALLS, FORCE, SPLIT), False)])
def test_tiles_of_half_the_threads(kind, pair):
    L = need_gpu()
    banner(f"pairs {kind}")
    s = _solver(L, 9, (1, 545, 513), kind)  # 306 tiles of 32
    names = _kernels(lambda: s.step(8))
    s.close()
    assert (MULTI + "<32" in names) and (", true>" in names.split(MULTI)[1]) == pair, names
