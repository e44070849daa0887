"""vlasov_step_moments on the blocks whose last kick sums the moments
otherwise than the cubic ones of 16 and 32 do.

64^3 blocks: while the uy-uz kernel stores its eight slabs per cell, on fewer
cells than work-groups and on more (294 against 256 CUs, one work-group each:
sums published from one cell to the next).  33 x 40 x 32: larger than LDS, so
the last kick is three sweeps and a pass over the result.  f, its scales and
the outflow are vlasov_step's bits, and the moments those of vlasov_moments on
the result up to the order of their FP64 sums: 262144 values of one sign (rho),
and for umean of both signs around a mean far below the velocities.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs an MI355X", allow_module_level=True)

from paper_2110_15867_amd import vlasov as V  # noqa: E402

SHAPES = [((2, 3, 2), (64, 64, 64)), ((7, 7, 6), (64, 64, 64)), ((3, 2, 4), (33, 40, 32))]


@pytest.mark.parametrize("prec", [V.F32, V.F16, V.BF16])
@pytest.mark.parametrize("n,nu", SHAPES)
def test_step_moments_route(n, nu, prec):
    print("case: step moments route", n, nu, V.PREC_NAME[prec], flush=True)
    hg = V.make_grid(n, nu, (1.0, 1.3, 0.8), (1.0, 0.9, 1.1))
    gen = torch.Generator(device="cuda").manual_seed(29)
    f = torch.rand(V.grid_shape(hg), generator=gen, device="cuda") ** 2
    f *= torch.rand(tuple(n) + (1, 1, 1), generator=gen, device="cuda") + 0.5   # cells differ
    st = V.encode(hg, prec, f)
    gs = [torch.rand((3,) + n, generator=gen, device="cuda") * 6 - 3 for _ in range(2)]
    o1 = torch.zeros(n, dtype=torch.float64, device="cuda")
    o2 = torch.zeros_like(o1)
    ref = V.step(st, gs[0], gs[1], 0.17, outflow=o1)
    nb = V.vlasov_step_workspace_bytes(hg, prec)
    work = torch.empty(nb, dtype=torch.uint8, device="cuda")
    out = V.empty_state(hg, prec, "cuda")
    rho = torch.full(n, np.nan, dtype=torch.float64, device="cuda")
    um = torch.full((3,) + n, np.nan, dtype=torch.float64, device="cuda")
    V.vlasov_step_moments(hg, prec, V.VBC_OUTFLOW, st.f, st.scale, out.f, out.scale, gs[0], gs[1],
                          0.17, 1.0, work, nb, o2, rho, um)
    assert torch.equal(out.f, ref.f)
    if prec != V.F32:
        assert torch.equal(out.scale, ref.scale)
    assert torch.equal(o1, o2)
    rho_k, um_k, _ = V.moments(out)
    # FP64 sums in two orders: at most 262144 roundings each, far fewer through
    # the trees; umean relative to the largest velocity (its terms' size)
    np.testing.assert_allclose(rho.cpu().numpy(), rho_k.cpu().numpy(), rtol=1e-12, atol=0)
    np.testing.assert_allclose(um.cpu().numpy(), um_k.cpu().numpy(), rtol=0, atol=1e-12)
    # and without umean
    rho2 = torch.full_like(rho, np.nan)
    V.vlasov_step_moments(hg, prec, V.VBC_OUTFLOW, st.f, st.scale, out.f, out.scale, gs[0], gs[1],
                          0.17, 1.0, work, nb, None, rho2, None)
    assert torch.equal(rho2, rho)
