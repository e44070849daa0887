"""The fused kick of block shapes without a kernel of their own.

vlasov_kick on such a block gives the bits of vlasov_advect_ux, _uy, _uz in
sequence, in every storage form: line lengths around the walk's groups of
four cells (1 to 9, 13, 64, 65), one-cell axes, uz-lines loaded by 1, 2 and 4
values, the largest block that fits LDS and one beyond it (the three single
sweeps), both velocity boundaries, shifts beyond the block.  The outflow of a
cell sums FP32 line values grouped differently: 1e-6 relative, as for the
cubic blocks.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs an MI355X", allow_module_level=True)

from paper_2110_15867_amd import vlasov as V  # noqa: E402

SHAPES = [(1, 1, 1), (1, 2, 3), (2, 1, 5), (4, 3, 2), (5, 6, 7), (9, 8, 4), (6, 1, 13),
          (24, 20, 18), (65, 3, 4), (3, 64, 5), (2, 3, 65), (40, 30, 30), (40, 36, 30)]
SCALED = [(1, 1, 4), (3, 5, 8), (9, 13, 16), (6, 65, 4), (2, 3, 64), (20, 30, 32), (33, 40, 32)]


def _compare(nu, prec, vbc, cfl):
    print("case: any kick", nu, V.PREC_NAME[prec], vbc, cfl, flush=True)
    n = (3, 2, 3)
    hg = V.make_grid(n, nu, (1.0, 1.0, 1.0), (1.0, 0.9, 1.1))
    rng = np.random.default_rng(abs(hash((nu, prec, vbc))) % 10000)
    f = rng.uniform(0, 1, V.grid_shape(hg)).astype(np.float32) ** 2
    f[rng.uniform(size=f.shape) < 0.2] = 0.0
    st = V.encode(hg, prec, torch.from_numpy(f).cuda())
    dt = 0.1
    field = np.stack([rng.uniform(-cfl, cfl, n) * 2 * hg.umax[a] / nu[a] / dt for a in range(3)])
    field[:, 0, 0, 0] = 0.0
    g = torch.from_numpy(field.astype(np.float32)).cuda()
    o1 = torch.ones(n, dtype=torch.float64, device="cuda")
    o2 = torch.ones(n, dtype=torch.float64, device="cuda")
    a = st
    for ax in ("ux", "uy", "uz"):
        a = V.advect(ax, a, dt, g=g, vbc=vbc, outflow=o1)
    k = V.kick(st, g, dt, vbc=vbc, outflow=o2)
    assert torch.equal(k.f, a.f)
    if prec != V.F32:
        assert torch.equal(k.scale, a.scale)
    np.testing.assert_allclose(o2.cpu().numpy(), o1.cpu().numpy(), rtol=1e-6, atol=0)


@pytest.mark.parametrize("nu", SHAPES)
@pytest.mark.parametrize("vbc", [V.VBC_OUTFLOW, V.VBC_PERIODIC])
@pytest.mark.parametrize("cfl", [0.9, 70.0])
def test_any_kick_equals_three_sweeps(nu, vbc, cfl):
    _compare(nu, V.F32, vbc, cfl)


@pytest.mark.parametrize("nu", SCALED)
@pytest.mark.parametrize("prec", [V.F16, V.BF16])
@pytest.mark.parametrize("vbc", [V.VBC_OUTFLOW, V.VBC_PERIODIC])
def test_any_kick_equals_three_scaled_sweeps(nu, prec, vbc):
    _compare(nu, prec, vbc, 3.3)


def test_any_kick_still_needs_a_workspace():
    hg = V.make_grid((2, 2, 2), (8, 6, 4))
    f = torch.rand(V.grid_shape(hg), device="cuda")
    g = torch.zeros((3, 2, 2, 2), device="cuda")
    with pytest.raises(V.VlasovError):
        V.vlasov_kick(hg, V.F32, V.VBC_OUTFLOW, f, None, torch.empty_like(f), None, g, 0.1)
