"""Every route of the position sweeps on a grid that reaches it.

Small grids take one line per thread and lines of 16 and 32 cells the LDS
tiles, so the walks of four and two lines per thread, the gathered y waves and
the paired z walk each need a grid of their own; position_route restates the
host's rules and each case says which route it is for.  FP32: the bits of the
sweep of the transposed grid along another axis, whose walk is another one.
FP16/BF16: the codes and scales of that FP32 sweep of the decoded values.
"""
import pytest

from route_rules import position_route

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs an MI355X", allow_module_level=True)

from paper_2110_15867_amd import vlasov as V  # noqa: E402

PERM = {("x", "z"): (1, 2, 0), ("y", "z"): (0, 2, 1), ("y", "x"): (1, 0, 2), ("z", "x"): (2, 0, 1)}


def _check(axis, other, n, nu, prec, shift, route):
    k = "xyz".index(axis)
    print("case: route", route, axis, n, nu, V.PREC_NAME[prec], shift, flush=True)
    top = 1 - 1 / nu[k]                               # largest |u| at a cell centre
    assert position_route(n, nu, k, prec != V.F32, abs(shift), shift > 0) == route
    perm = PERM[axis, other]
    g = V.make_grid(n, nu)
    t = V.make_grid(tuple(n[p] for p in perm), tuple(nu[p] for p in perm))
    full = perm + tuple(3 + p for p in perm)
    back = sorted(range(6), key=full.__getitem__)
    gen = torch.Generator(device="cuda").manual_seed(n[k] + nu[2])
    f = torch.rand(V.grid_shape(g), generator=gen, device="cuda") ** 2
    f[torch.rand(f.shape, generator=gen, device="cuda") < 0.2] = 0.0
    st = V.encode(g, prec, f)
    dt = shift / n[k] / top
    got = V.advect(axis, st, dt)
    want = V.advect(other, V.State(t, V.F32, V.decode(st).permute(full).contiguous()), dt)
    want = V.encode(g, prec, want.f.permute(back).contiguous())
    assert torch.equal(got.f, want.f)
    if prec != V.F32:
        assert torch.equal(got.scale, want.scale)


@pytest.mark.parametrize("axis", ["x", "y"])
@pytest.mark.parametrize("nu", [(24, 20, 18), (6, 5, 90)])
@pytest.mark.parametrize("ny", [20, 16])
@pytest.mark.parametrize("shift", [0.4, 2.5, -1.7])
def test_two_lines_per_thread(axis, nu, ny, shift):
    _check(axis, "z", (16 if ny == 16 else 6, ny, 18), nu, V.F32, shift, ("walk", 2))


# waves of eight u_y (whose count gathered waves do not take), one or more
# integer parts per wave; FP16/BF16 lines of 64 cells stay out of the tiles
@pytest.mark.parametrize("ny", [16, 32, 64, 20])
@pytest.mark.parametrize("shift", [0.6, 1.4, 2.6, -1.4])
def test_consecutive_y_waves(ny, shift):
    _check("y", "x", (8, ny, 8), (8, 18, 32), V.F32, shift, ("walk", 4))


@pytest.mark.parametrize("prec", [V.F16, V.BF16])
@pytest.mark.parametrize("ny,nu", [(64, (8, 18, 32)), (20, (8, 18, 32)), (32, (8, 72, 8))])
@pytest.mark.parametrize("shift", [0.6, 2.6, -1.4])
def test_consecutive_y_waves_scaled(prec, ny, nu, shift):
    _check("y", "x", (8, ny, 8), nu, prec, shift, ("walk", 4))


@pytest.mark.parametrize("prec", [V.F32, V.F16, V.BF16])
@pytest.mark.parametrize("ny", [16, 32, 64, 20])
@pytest.mark.parametrize("shift", [0.6, 2.6, -1.4])
def test_gathered_y_waves(prec, ny, shift):
    _check("y", "x", (8, ny, 8), (8, 8, 64), prec, shift, ("gathered", 4))


@pytest.mark.parametrize("prec", [V.F16, V.BF16])
@pytest.mark.parametrize("n,nu", [((2, 3, 64), (4, 8, 16)), ((3, 2, 64), (4, 4, 32)),
                                  ((2, 2, 64), (2, 2, 64)), ((1, 1, 64), (2, 4, 16))])
@pytest.mark.parametrize("shift", [0.05, 0.6, 0.98])
def test_paired_z_walk(prec, n, nu, shift):
    _check("z", "x", n, nu, prec, shift, ("pair", 1))
