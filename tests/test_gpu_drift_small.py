"""The three drifts of a small mesh in one pass (FP32 steps): the bits of the
single sweeps.

vlasov_step and vlasov_steps against the chain vlasov_kick, vlasov_advect_z,
_y, _x, vlasov_kick for every mix of sides of 8 and 16, one work-group of u_z
values and several, groups of 32 tiles (placed by line) and other counts, and
shapes the pass leaves to the others; fractional, whole-cell, multi-cell, zero
and reversed shifts.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs an MI355X", allow_module_level=True)

from paper_2110_15867_amd import vlasov as V  # noqa: E402

SHAPES = [((a, b, c), (4, 6, 16)) for a in (8, 16) for b in (8, 16) for c in (8, 16)]
SHAPES += [((8, 8, 8), (1, 1, 8)), ((8, 16, 8), (3, 5, 24)), ((16, 8, 16), (8, 8, 32)),
           ((8, 8, 16), (5, 2, 40)), ((8, 16, 16), (16, 16, 16)), ((8, 8, 8), (16, 32, 32)),
           # left to the other passes
           ((8, 8, 8), (4, 4, 12)), ((8, 12, 8), (4, 4, 16)), ((8, 8, 32), (4, 4, 16)),
           ((8, 8, 16), (16, 16, 40))]


def chain(st, gs, hs, dt):
    st = V.kick(st, gs[0], hs[0])
    for g, h in zip(gs[1:], hs[1:]):
        for ax in ("z", "y", "x"):
            st = V.advect(ax, st, dt)
        st = V.kick(st, g, h)
    return st


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("dt", [0.0, 0.043, 0.31, -0.17, 1.9])
def test_step_is_the_chain_of_single_launches(shape, dt):
    n, nu = shape
    print("case: small drifts", n, nu, dt, flush=True)
    hg = V.make_grid(n, nu, (1.0, 1.3, 0.8), (1.0, 0.9, 1.1))
    rng = np.random.default_rng(sum(n) * 7 + sum(nu))
    f = rng.uniform(0, 1, V.grid_shape(hg)).astype(np.float32) ** 2
    f[rng.uniform(size=f.shape) < 0.1] = 0.0
    st = V.State(hg, V.F32, torch.from_numpy(f).cuda())
    gs = [torch.from_numpy(rng.uniform(-3, 3, (3,) + n).astype(np.float32)).cuda() for _ in range(3)]
    h = 0.5 * dt
    got = V.step(st, gs[0], gs[1], dt)
    assert torch.equal(got.f, chain(st, gs[:2], (h, h), dt).f)
    out = V.empty_state(hg, V.F32, "cuda")
    nb = V.vlasov_steps_workspace_bytes(hg, V.F32)
    work = torch.empty(nb, dtype=torch.uint8, device="cuda")
    V.vlasov_steps(hg, V.F32, V.VBC_OUTFLOW, st.f, None, out.f, None, torch.stack(gs).contiguous(),
                   2, dt, None, work, nb, None)
    assert torch.equal(out.f, chain(st, gs, (h, dt, h), dt).f)
