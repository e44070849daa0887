"""The z sweep through LDS tiles: the bits of the other walks.

FP32: a z sweep equals the x sweep of the transposed grid (another kernel) bit
for bit, whatever the shift: below a cell, several cells, whole turns of the
box, whole cells, none, either direction; line lengths 16, 32 and 64 (the last
one from HBM where no line moves by a cell), uz-lines of 16, 32 and 64 values,
rows of one wave and of many, a wave count that does not fill the last
work-group, and beside them lengths and uz-lines the tiles do not take.
FP16/BF16: the codes and scales of the FP32 sweep of the decoded values.
"""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs an MI355X", allow_module_level=True)

from paper_2110_15867_amd import vlasov as V  # noqa: E402

GRIDS = [((1, 1, 16), (2, 2, 16)), ((3, 1, 16), (1, 5, 64)), ((2, 3, 32), (3, 4, 32)),
         ((1, 3, 32), (4, 3, 16)), ((1, 2, 64), (2, 3, 32)), ((2, 1, 64), (1, 7, 64)),
         ((2, 2, 24), (2, 2, 32)), ((2, 2, 32), (2, 4, 8)), ((1, 2, 16), (1, 1, 16))]


@pytest.mark.parametrize("grid", GRIDS)
@pytest.mark.parametrize("cfl", [0.0, 0.4, 0.999, 2.5, -1.7, 16.0, 37.3])
def test_z_tiles(grid, cfl):
    n, nu = grid
    print("case: z tiles", n, nu, cfl, flush=True)
    M = n[2]
    gz = V.make_grid(n, nu, (1.0, 1.0, 1.0), (1.0, 1.0, 0.9))
    gx = V.make_grid((M, n[0], n[1]), (nu[2], nu[0], nu[1]), (1.0, 1.0, 1.0), (0.9, 1.0, 1.0))
    gen = torch.Generator(device="cuda").manual_seed(M + nu[2])
    f = torch.rand(V.grid_shape(gz), generator=gen, device="cuda") ** 2
    f[torch.rand(f.shape, generator=gen, device="cuda") < 0.2] = 0.0
    dt = cfl / M
    z = V.advect("z", V.State(gz, V.F32, f), dt)
    x = V.advect("x", V.State(gx, V.F32, f.permute(2, 0, 1, 5, 3, 4).contiguous()), dt)
    assert torch.equal(z.f, x.f.permute(1, 2, 0, 4, 5, 3))
    for prec in (V.F16, V.BF16):
        st = V.encode(gz, prec, f)
        got = V.advect("z", st, dt)
        want = V.encode(gz, prec, V.advect("z", V.State(gz, V.F32, V.decode(st)), dt).f)
        assert torch.equal(got.f, want.f)
        assert torch.equal(got.scale, want.scale)
