"""The gradient run inside a captured graph: every replay, with new inputs in
its buffers and eager work in between, gives the eager gradients."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs an MI355X", allow_module_level=True)

from paper_2110_15867_amd import autograd as A  # noqa: E402
from paper_2110_15867_amd import vlasov as V  # noqa: E402


@pytest.mark.parametrize("n,nu,modes", [((8, 8, 8), (8, 8, 8), 4), ((32, 32, 32), (4, 4, 4), 1)])
def test_replays_give_the_eager_gradients(n, nu, modes):
    print("case: gradient capture", n, nu, modes, flush=True)
    grid, steps = V.make_grid(n, nu), 2
    gen = torch.Generator(device="cuda").manual_seed(1)

    def rand(*shape, dtype=torch.float32):
        return torch.rand(shape, generator=gen, device="cuda", dtype=dtype)

    problem = A.RunProblem(grid, [rand(modes, 3, *n) - 0.5 for _ in range(steps + 1)], 0.02, steps)
    f = rand(*V.grid_shape(grid)).requires_grad_()
    B = rand(modes, dtype=torch.float64).requires_grad_()
    lam = rand(*n, dtype=torch.float64)

    def gradients():
        return torch.autograd.grad(A.VlasovRun.apply(f, B, problem), (f, B), lam)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        gradients()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = gradients()
    for _ in range(4):
        with torch.no_grad():
            f.copy_(rand(*f.shape))
            B.copy_(rand(modes, dtype=torch.float64))
        want = [w.clone() for w in gradients()]
        float(rand(1 << 20).sum())
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(out, want):
            assert torch.equal(a, b)
