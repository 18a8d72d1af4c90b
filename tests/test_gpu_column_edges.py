"""The column kernels on grids large enough for them (column_pays) with sides of one
node and few planes: bitwise the one-thread-per-node kernels (variant GENERIC).
Which kernel runs is test_gpu_routes.py's."""
import pytest
import torch

from gpu_helpers import banner, need_gpu

pytestmark = pytest.mark.gpu

GENERIC = 1
WIDE = [(4, 1, 90001), (4, 90001, 1), (5, 300, 301), (9, 211, 97), (90, 75, 75)]


def _solver(L, shape, kind, variant):
    nz, ny, nx = shape
    gen = torch.Generator(device="cuda")
    gen.manual_seed(221)
    kw = {}
    if "walls" in kind:
        m = (torch.rand(shape, device="cuda", generator=gen) < 0.03).to(torch.uint8)
        kw = dict(mask=m, wall_u=[[0.0] * 3, [0.03, 0.01, -0.02]])
    if "force" in kind:
        kw["g"] = (1e-5, -2e-6, 3e-6)
    s = L.Solver(19, nx, ny, nz, 1.7, storage=1 if "fp16" in kind else 0, variant=variant,
                 fp16_rounding=(0, 0) if "nearest" in kind else None, **kw)
    u = 0.02 * torch.randn((3,) + shape, device="cuda", generator=gen)
    if "field" in kind:
        s.set_force_field(1e-3 * u)
    s.set_state(0.1 * u[0], u)
    return s


@pytest.mark.parametrize("shape,kind", [(s, k) for s in WIDE for k in ("plain", "force", "field",
                                                                       "walls", "walls fp16")] +
                         [(WIDE[-1], "fp16"), (WIDE[-1], "fp16 nearest"), ((4, 1, 90001), "fp16"),
                          ((1, 1, 300), "walls"), ((5, 1, 511), "walls"), ((2, 401, 3), "walls")])
def test_columns_with_sides_of_one_node(shape, kind):
    L = need_gpu()
    banner(f"column edges {shape} {kind}")
    a, b = _solver(L, shape, kind, 0), _solver(L, shape, kind, GENERIC)
    for steps in (1, 3):
        a.step(steps)
        b.step(steps)
        assert torch.equal(a.save_state(), b.save_state()), steps
        (ma, ea), (mb, eb) = a.diagnostics(), b.diagnostics()
        assert abs(ma - mb) <= 1e-12 * abs(mb) and abs(ea - eb) <= 1e-12 * abs(eb)
    a.close()
    b.close()


@pytest.mark.parametrize("shape", WIDE)
@pytest.mark.parametrize("t0", [0, 5])
def test_reverse_columns(shape, t0):
    L = need_gpu()
    banner(f"reverse column edges {shape} t0={t0}")
    s = _solver(L, shape, "plain", 0)
    st = s.save_state()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(223)
    mu = torch.randn(shape + (4,), device="cuda", generator=gen)
    out = []
    for variant in (0, GENERIC):
        L.lwacm_set_variant(s.ctx, variant)
        mo = torch.empty_like(mu)
        dw = torch.zeros(1, dtype=torch.float64, device="cuda")
        L.lwacm_adjoint_step(s.ctx, st, mu, mo, dw, t0 == 0)
        out.append((mo, float(dw)))
    s.close()
    (a, wa), (b, wb) = out
    assert torch.equal(a, b) and abs(wa - wb) <= 1e-12 * abs(wb) + 1e-12
