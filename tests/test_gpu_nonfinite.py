"""Sweeps of data that hold NaN or infinities: every route gives the values of
the general one.

A NaN spreads along its own line, as far as the stencils that read it, and
with FP16/BF16 storage it is left out of the scale of its uz-line: the other
values of that line keep theirs.  An infinity is the scale of its uz-line.
Compared value by value, with NaN in the same places: the y and z sweeps
(lines through LDS tiles and others) with the x sweep of the transposed grid,
encoded; a kick of a block held in LDS with its three single sweeps; the fused
drifts of a step with the single sweeps.  Four neighbouring values along u_z
(the values of one lane of a row) are corrupted together, or one.
"""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs an MI355X", allow_module_level=True)

from paper_2110_15867_amd import vlasov as V  # noqa: E402


def _same(a, b):
    assert torch.equal(torch.isnan(a), torch.isnan(b))
    assert torch.equal(a.nan_to_num(nan=0.0), b.nan_to_num(nan=0.0))


def _corrupt(f, bad, gen):
    """Groups of four values along u_z, and single ones, set to `bad`."""
    lines = f.view(-1, f.shape[-1])
    for k in range(8):
        l = int(torch.randint(lines.shape[0], (1,), generator=gen))
        j = 4 * int(torch.randint(lines.shape[1] // 4, (1,), generator=gen))
        lines[l, j:j + (4 if k % 2 else 1)] = bad
    return f


def _data(grid, seed):
    gen = torch.Generator().manual_seed(seed)
    return torch.rand(V.grid_shape(grid), generator=gen).cuda() ** 2, gen


GRIDS = [("y", (2, 16, 2), (4, 4, 16)), ("y", (2, 32, 1), (4, 4, 32)), ("y", (1, 64, 2), (2, 4, 16)),
         ("z", (2, 2, 16), (4, 4, 16)), ("z", (2, 1, 32), (4, 4, 32)), ("z", (1, 2, 64), (2, 4, 64)),
         ("z", (1, 2, 20), (4, 4, 16))]


@pytest.mark.parametrize("case", GRIDS)
@pytest.mark.parametrize("prec", [V.F32, V.F16, V.BF16])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("cfl", [0.4, 2.5])
def test_position_sweeps(case, prec, bad, cfl):
    axis, n, nu = case
    print("case: nonfinite", axis, n, nu, V.PREC_NAME[prec], bad, cfl, flush=True)
    k = "xyz".index(axis)
    perm = (1, 0, 2) if k == 1 else (2, 0, 1)          # that axis first
    perm = perm + tuple(3 + p for p in perm)
    back = sorted(range(6), key=perm.__getitem__)
    g = V.make_grid(n, nu)
    gx = V.make_grid(tuple(n[p] for p in perm[:3]), tuple(nu[p] for p in perm[:3]))
    f, gen = _data(g, 5)
    st = V.encode(g, prec, f)
    _corrupt(st.f, bad, gen)
    dt = cfl / n[k]
    got = V.advect(axis, st, dt)
    x = V.advect("x", V.State(gx, V.F32, V.decode(st).permute(perm).contiguous()), dt)
    want = V.encode(g, prec, x.f.permute(back).contiguous())
    assert torch.isfinite(got.f).any() and not torch.isfinite(got.f).all()
    _same(got.f, want.f)
    if prec != V.F32:
        _same(got.scale, want.scale)


@pytest.mark.parametrize("nu", [(8, 6, 16), (9, 13, 4)])
@pytest.mark.parametrize("prec", [V.F32, V.F16, V.BF16])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_kick_of_a_block_in_lds(nu, prec, bad):
    print("case: nonfinite kick", nu, V.PREC_NAME[prec], bad, flush=True)
    n = (3, 2, 2)
    g = V.make_grid(n, nu)
    f, gen = _data(g, 6)
    st = V.encode(g, prec, f)
    _corrupt(st.f, bad, gen)
    field = (torch.rand((3,) + n, generator=gen) * 6 - 3).cuda()
    want = st
    for ax in ("ux", "uy", "uz"):
        want = V.advect(ax, want, 0.07, g=field)
    got = V.kick(st, field, 0.07)
    assert torch.isfinite(got.f).any() and not torch.isfinite(got.f).all()
    _same(got.f, want.f)
    if prec != V.F32:
        _same(got.scale, want.scale)


# drifts of a small mesh in one launch; y and x in one pass
@pytest.mark.parametrize("grid", [((8, 8, 8), (8, 8, 8)), ((8, 9, 4), (32, 32, 16))])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_fused_drifts(grid, bad):
    n, nu = grid
    print("case: nonfinite drifts", n, nu, bad, flush=True)
    g = V.make_grid(n, nu)
    f, gen = _data(g, 7)
    _corrupt(f, bad, gen)
    st = V.State(g, V.F32, f)
    field = (torch.rand((3,) + n, generator=gen) * 2 - 1).cuda()
    want = V.kick(st, field, 0.05)
    for ax in ("z", "y", "x"):
        want = V.advect(ax, want, 0.1)
    want = V.kick(want, field, 0.05)
    got = V.step(st, field, field, 0.1)
    assert torch.isfinite(got.f).any() and not torch.isfinite(got.f).all()
    _same(got.f, want.f)
