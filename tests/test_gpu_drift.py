"""The y and x drifts in one pass (FP32 steps): the bits of the single sweeps.

vlasov_step against the chain vlasov_kick, vlasov_advect_z, _y, _x,
vlasov_kick on the shapes where the fused pass can go wrong: y-lines of one
segment, with an overlapping last segment, of every segment length (5 to 8
cells) and of sixteen segments; x-lines from the shortest taken (8) around
the walk's groups of five planes; z cells that do not fill a wave, uz-lines
beyond a wave; shapes it leaves to the single sweeps; fractional, whole-cell, multi-cell, zero and reversed shifts.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs an MI355X", allow_module_level=True)

from paper_2110_15867_amd import vlasov as V  # noqa: E402

# the fused pass is taken from 2048 waves on
SHAPES = [((9, 8, 8), (32, 32, 16)), ((8, 9, 4), (32, 32, 16)), ((13, 10, 4), (16, 64, 16)),
          ((10, 12, 4), (32, 32, 32)), ((11, 14, 2), (16, 32, 64)), ((8, 15, 5), (32, 32, 16)),
          ((12, 33, 2), (16, 32, 32)), ((64, 8, 2), (32, 64, 64)), ((9, 128, 1), (8, 16, 64)),
          ((8, 16, 2), (16, 16, 128)),
          # segments of 5 cells below 4096 waves; the same lines above
          ((9, 8, 8), (64, 32, 16)), ((10, 12, 4), (64, 32, 32)), ((11, 14, 2), (32, 64, 64)),
          ((8, 15, 5), (64, 32, 16)), ((8, 16, 2), (32, 16, 128)), ((8, 80, 1), (8, 16, 64)),
          # left to the single sweeps
          ((8, 129, 1), (8, 16, 64)), ((7, 16, 4), (32, 32, 16)), ((16, 7, 8), (32, 32, 16)),
          ((8, 16, 4), (32, 32, 8)), ((8, 16, 4), (3, 5, 16))]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("dt", [0.0, 0.043, 0.31, -0.17, 1.9])
def test_step_is_the_chain_of_single_launches(shape, dt):
    n, nu = shape
    print("case: fused drifts", n, nu, dt, flush=True)
    hg = V.make_grid(n, nu, (1.0, 1.3, 0.8), (1.0, 0.9, 1.1))
    rng = np.random.default_rng(sum(n) * 7 + sum(nu))
    f = rng.uniform(0, 1, V.grid_shape(hg)).astype(np.float32) ** 2
    f[rng.uniform(size=f.shape) < 0.1] = 0.0
    st = V.State(hg, V.F32, torch.from_numpy(f).cuda())
    gs = [torch.from_numpy(rng.uniform(-3, 3, (3,) + n).astype(np.float32)).cuda() for _ in range(2)]
    ref = V.kick(st, gs[0], 0.5 * dt)
    for ax in ("z", "y", "x"):
        ref = V.advect(ax, ref, dt)
    ref = V.kick(ref, gs[1], 0.5 * dt)
    got = V.step(st, gs[0], gs[1], dt)
    assert torch.equal(got.f, ref.f)
    # several steps, through vlasov_steps' buffers
    out = V.empty_state(hg, V.F32, "cuda")
    nb = V.vlasov_steps_workspace_bytes(hg, V.F32)
    work = torch.empty(nb, dtype=torch.uint8, device="cuda")
    fields = torch.stack(gs + gs[:1]).contiguous()
    V.vlasov_steps(hg, V.F32, V.VBC_OUTFLOW, st.f, None, out.f, None, fields, 2, dt, None, work,
                   nb, None)
    ref = V.kick(st, gs[0], 0.5 * dt)
    for k, h in ((1, dt), (0, 0.5 * dt)):
        for ax in ("z", "y", "x"):
            ref = V.advect(ax, ref, dt)
        ref = V.kick(ref, gs[k], h)
    assert torch.equal(out.f, ref.f)


def test_whole_cell_drift_is_a_translation():
    """u dt / dx a whole number in every velocity cell: the step permutes."""
    hg = V.make_grid((8, 16, 8), (16, 16, 16), (1.0, 1.0, 1.0), (1.0, 1.0, 1.0))
    gen = torch.Generator(device="cuda").manual_seed(3)
    f = torch.rand(V.grid_shape(hg), generator=gen, device="cuda")
    g = torch.zeros((3, 8, 16, 8), device="cuda")
    # u = (2 j - 15) / 16; dt = 2: x and z shifts of 16 u = 2 j - 15, y of twice that
    got = V.step(V.State(hg, V.F32, f), g, g, 2.0)
    want = torch.empty_like(f)
    for jx in range(16):
        for jy in range(16):
            for jz in range(16):
                s = [2 * j - 15 for j in (jx, jy, jz)]
                want[..., jx, jy, jz] = torch.roll(f[..., jx, jy, jz], (s[0], 2 * s[1], s[2]),
                                                   (0, 1, 2))
    assert torch.equal(got.f, want)
