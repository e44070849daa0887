"""The outflow tally of kicks of blocks held whole in LDS, at any shift.

A single sweep sums what a group of lines loses in FP32, row by row: the first
two rows past the face, the flux through it, then the rows further out.  The
fused kick adds the same values in the same order, so a cell's tally is that
of vlasov_advect_ux, _uy, _uz up to its FP64 sums, whose order differs: below
4096 terms of one sign per sweep, 4096 * 2^-53 * 3 = 1.4e-12 relative at the
very most.  Shifts of less than a cell, of three and more (rows further out),
of the block's length and beyond; uz-lines taken by 1, 2 and 4 lines at a time.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs an MI355X", allow_module_level=True)

from paper_2110_15867_amd import vlasov as V  # noqa: E402


@pytest.mark.parametrize("nu", [(5, 6, 7), (9, 8, 6), (6, 1, 13), (1, 9, 4), (24, 20, 16), (9, 13, 16)])
@pytest.mark.parametrize("prec", [V.F32, V.F16, V.BF16])
@pytest.mark.parametrize("cells", [0.9, 2.5, 5.5, 30.0])
def test_outflow_of_the_three_sweeps(nu, prec, cells):
    if prec != V.F32 and nu[2] & (nu[2] - 1):
        pytest.skip("no scaled storage for this uz-line")
    print("case: kick outflow", nu, V.PREC_NAME[prec], cells, flush=True)
    n, dt = (4, 3, 3), 0.1
    hg = V.make_grid(n, nu, (1.0, 1.0, 1.0), (1.0, 0.9, 1.1))
    rng = np.random.default_rng(sum(nu))
    f = rng.uniform(0, 1, V.grid_shape(hg)).astype(np.float32) ** 2
    st = V.encode(hg, prec, torch.from_numpy(f).cuda())
    s = rng.uniform(-cells, cells, (3,) + n)
    g = np.stack([s[a] * 2 * hg.umax[a] / nu[a] / dt for a in range(3)]).astype(np.float32)
    gt = torch.from_numpy(g).cuda()
    want = torch.zeros(n, dtype=torch.float64, device="cuda")
    got = torch.zeros_like(want)
    a = st
    for ax in ("ux", "uy", "uz"):
        a = V.advect(ax, a, dt, g=gt, outflow=want)
    k = V.kick(st, gt, dt, outflow=got)
    assert torch.equal(k.f, a.f)
    np.testing.assert_allclose(got.cpu().numpy(), want.cpu().numpy(), rtol=1.4e-12, atol=0)
