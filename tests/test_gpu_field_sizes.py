"""vlasov_field over mesh sizes: one-cell axes, primes (the any-radix step),
odd composites, every register radix, rows that do not fill a bundle of
lines, the longest lines transformed in LDS (256) and one beyond (257, the
direct sums).

Against the oracle's FP64 solve.  The result is FP32 and the FP64 transforms
add about 1e-15, so the bound is one FP32 rounding (2^-24 of a value, at most
the field's largest) plus as much again.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs an MI355X", allow_module_level=True)

from paper_2110_15867_amd import vlasov as V  # noqa: E402


@pytest.mark.parametrize("n", [(1, 1, 2), (1, 5, 8), (7, 1, 1), (2, 3, 17), (11, 13, 7),
                               (64, 48, 30), (21, 10, 35), (96, 2, 25), (3, 97, 4), (4, 3, 251),
                               (256, 4, 6), (5, 6, 256), (3, 192, 2), (257, 2, 3)])
def test_field_sizes(n):
    print("case: field", n, flush=True)
    L = (1.0, 1.7, 0.6)
    og = oracle.Grid.make(n, (4, 4, 4), L, (1, 1, 1))
    hg = V.make_grid(n, (4, 4, 4), L)
    rho = np.random.default_rng(hash(n) % 1000).uniform(0.5, 1.5, n)
    want = oracle.field_from_density(og, rho, -2.3)
    got = V.field(hg, torch.from_numpy(rho).cuda(), -2.3).double().cpu().numpy()
    assert np.abs(got - want).max() <= 2.0 ** -23 * np.abs(want).max() + 1e-30
