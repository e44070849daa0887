"""The y sweep through LDS tiles: the bits of the other walks.

As for z: an FP32 y sweep equals the x sweep of the transposed grid bit for
bit, and the FP16/BF16 codes and scales are those of the FP32 sweep of the
decoded values.  Lines of 16, 32 and 64 cells, uz-lines of 16 and 32 values
(and of 64 and 8, left to the other walks), u_y counts below, at and beyond
the lines of a wave and not dividing it, a wave count that does not fill the
last work-group, shifts below a cell (uz-lines of 32: from HBM), of several
cells, whole turns, whole cells, none, either direction.
"""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs an MI355X", allow_module_level=True)

from paper_2110_15867_amd import vlasov as V  # noqa: E402

GRIDS = [((1, 16, 1), (4, 1, 16)), ((3, 16, 1), (2, 6, 16)), ((2, 32, 3), (4, 3, 32)),
         ((1, 32, 3), (4, 3, 16)), ((1, 64, 2), (2, 10, 16)), ((2, 64, 1), (2, 5, 32)),
         ((2, 16, 1), (2, 1, 32)), ((1, 16, 2), (16, 8, 64)), ((2, 32, 2), (2, 4, 8)),
         ((2, 24, 2), (2, 2, 16))]


@pytest.mark.parametrize("grid", GRIDS)
@pytest.mark.parametrize("cfl", [0.0, 0.4, 0.999, 2.5, -1.7, 16.0, 37.3])
def test_y_tiles(grid, cfl):
    n, nu = grid
    print("case: y tiles", n, nu, cfl, flush=True)
    M = n[1]
    gy = V.make_grid(n, nu, (1.0, 1.0, 1.0), (1.0, 0.9, 1.0))
    gx = V.make_grid((M, n[0], n[2]), (nu[1], nu[0], nu[2]), (1.0, 1.0, 1.0), (0.9, 1.0, 1.0))
    gen = torch.Generator(device="cuda").manual_seed(M + nu[2])
    f = torch.rand(V.grid_shape(gy), generator=gen, device="cuda") ** 2
    f[torch.rand(f.shape, generator=gen, device="cuda") < 0.2] = 0.0
    dt = cfl / M
    y = V.advect("y", V.State(gy, V.F32, f), dt)
    x = V.advect("x", V.State(gx, V.F32, f.permute(1, 0, 2, 4, 3, 5).contiguous()), dt)
    assert torch.equal(y.f, x.f.permute(1, 0, 2, 4, 3, 5))
    for prec in (V.F16, V.BF16):
        st = V.encode(gy, prec, f)
        got = V.advect("y", st, dt)
        want = V.encode(gy, prec, V.advect("y", V.State(gy, V.F32, V.decode(st)), dt).f)
        assert torch.equal(got.f, want.f)
        assert torch.equal(got.scale, want.scale)
