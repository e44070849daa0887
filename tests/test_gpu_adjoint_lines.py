"""Adjoint sweeps against the tangent sweeps, line by line.

Tangent and adjoint are separate kernels with the same frozen linearisation,
so on every line <T v, w> = <v, A w> (position sweeps), and the adjoint is the
transpose of the matrix of the tangent (velocity sweeps).
Line lengths around the walk's groups of four interfaces and its five-row
window (1 to 6, 15 to 18, 33), whole-cell, zero and large shifts, both
velocity boundaries, data with zeros, plateaus and steps (ties of the
limiter's and the clamp's selections), and enough cells that a work-group
takes several of them with a ragged last group.

Position lines: both sides are sums of at most a few terms per cell of FP32
products; the bound is 1e-5 of the sums of magnitudes.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs an MI355X", allow_module_level=True)

from paper_2110_15867_amd import vlasov as V  # noqa: E402


def _data(shape, seed):
    """Random cells; a third of them zero, a third rounded to eighths."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    r = torch.rand(shape, generator=gen, device="cuda")
    pick = torch.rand(shape, generator=gen, device="cuda")
    f = torch.where(pick < 0.33, torch.zeros_like(r),
                    torch.where(pick < 0.66, torch.round(r * 8) / 8, r * r))
    v = torch.randn(shape, generator=gen, device="cuda")
    w = torch.randn(shape, generator=gen, device="cuda")
    return f, v, w


def _check(tv, w, v, aw, dims, what):
    tv, w, v, aw = (t.double() for t in (tv, w, v, aw))
    gap = ((tv * w).sum(dims) - (v * aw).sum(dims)).abs()
    size = (tv * w).abs().sum(dims) + (v * aw).abs().sum(dims)
    assert bool((gap <= 1e-5 * size + 1e-30).all()), (what, float((gap / (size + 1e-30)).max()))


@pytest.mark.parametrize("M", [1, 2, 3, 4, 5, 6, 15, 16, 17, 18, 33])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_position_lines(M, axis):
    n = [3, 2, 2]
    n[axis] = M
    for nu in ((4, 8, 16), (5, 3, 7), (64, 4, 1)):
        hg = V.make_grid(n, nu, (1.0, 1.0, 1.0), (1.0, 1.0, 1.0))
        for k, dt in enumerate((0.0, 0.31 / M, 4.0 / M * nu[axis], 3.7 / M, -0.9 / M)):
            print("case: position lines", M, axis, nu, dt, flush=True)
            f, v, w = _data(V.grid_shape(hg), 10 * M + k)
            tv, aw = torch.empty_like(f), torch.empty_like(f)
            ax = "xyz"[axis]
            getattr(V, f"vlasov_advect_{ax}_tan")(hg, f, v, tv, dt)
            getattr(V, f"vlasov_advect_{ax}_adj")(hg, f, w, aw, dt)
            _check(tv, w, v, aw, (axis,), (M, axis, nu, dt))


@pytest.mark.parametrize("M", [1, 2, 3, 4, 5, 6, 15, 16, 17, 18, 32, 33])
@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("vbc", [V.VBC_OUTFLOW, V.VBC_PERIODIC])
def test_velocity_lines(M, axis, vbc):
    """Element by element: the tangents of the M unit rows are the columns of
    J, and J^T w in FP64 is the adjoint.  An element sums at most eleven terms
    (the identity and five interfaces' weights times two values of w) whose
    weights stay below 6, each after up to four FP32 roundings: 11 x 6 x 4 x
    2^-24 = 1.6e-5 of the largest |w|."""
    nu = [3, 5, 4]
    nu[axis] = M
    n = (17, 16, 17)                       # 4624 cells: two per work-group
    hg = V.make_grid(n, nu, (1.0, 1.0, 1.0), (1.0, 1.0, 1.0))
    print("case: velocity lines", M, axis, vbc, flush=True)
    f, v, w = _data(V.grid_shape(hg), 100 + M)
    gen = torch.Generator(device="cuda").manual_seed(M)
    s = (torch.rand((3,) + n, generator=gen, device="cuda") * 2 - 1) * 3.0
    s = torch.where(torch.rand(s.shape, generator=gen, device="cuda") < 0.2, torch.round(s), s)
    s[:, 0, 0, :4] = torch.tensor([0.0, 50.0, -50.0, 1e-7], device="cuda")
    dt = 0.25
    g = (s * (2.0 / M) / dt).float().contiguous()
    ax = "xyz"[axis]
    tan, adj = getattr(V, f"vlasov_advect_u{ax}_tan"), getattr(V, f"vlasov_advect_u{ax}_adj")
    tv, aw = torch.empty_like(f), torch.empty_like(f)
    lam_g = torch.zeros_like(g)
    adj(hg, vbc, f, g, dt, w, aw, lam_g)
    want = torch.empty(f.shape, dtype=torch.float64, device="cuda")
    for r in range(M):
        v.zero_()
        v.select(3 + axis, r).fill_(1.0)
        tan(hg, vbc, f, g, None, dt, v, tv)
        want.select(3 + axis, r).copy_((tv.double() * w.double()).sum(3 + axis))
    assert float((aw.double() - want).abs().max()) <= 1.6e-5 * float(w.abs().max())
    # the same cells in a grid small enough for one cell per work-group
    h1 = V.make_grid((1,) + n[1:], nu, (1.0 / 17, 1.0, 1.0), (1.0, 1.0, 1.0))
    a1 = torch.empty_like(f[5:6])
    l1 = torch.zeros((3, 1) + n[1:], device="cuda")
    adj(h1, vbc, f[5:6].contiguous(), g[:, 5:6].contiguous(), dt, w[5:6].contiguous(), a1, l1)
    assert torch.equal(a1, aw[5:6])
    assert torch.equal(l1, lam_g[:, 5:6])
