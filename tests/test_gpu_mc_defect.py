"""Monte Carlo on links that a load accepts but that are SU(3) only to about
8e-11 (the limit is 1e-10): the staples are products of the stored links, all
rows of them, so the chain follows the oracle's, which multiplies the same
matrices.  The bar is that of the Monte Carlo parity tests: ten times the
oracle's own divergence under a rotation by one rounding, at least 1e-11."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import oracle                                      # noqa: E402
from paper_2107_03747_amd import gen, tgf          # noqa: E402


@pytest.mark.parametrize("dims,twist", [((4, 4, 6, 8), tgf.PAPER_TWIST),
                                        ((6, 6, 4, 4), (1, 2, 1, 2, 1, 2))])
@pytest.mark.parametrize("n_or", [0, 1])
def test_mc_on_links_with_a_defect(dims, twist, n_or):
    rng = np.random.default_rng(12)
    U = gen.near_identity(dims, 0.3, seed=8).numpy()
    U = np.ascontiguousarray(U + 2e-11 * (rng.uniform(-1, 1, U.shape) +
                                          1j * rng.uniform(-1, 1, U.shape)))
    a = U.copy()
    b = np.ascontiguousarray(gen.near_identity(dims, 1e-15, seed=5).numpy() @ U)
    for x in (a, b):
        oracle.mc(x, dims, 0.5, 1, n_or, 99, twist=twist)
    bar = max(1e-11, 10 * float(np.abs(a - b).max()))
    f = tgf.Flow([(dims, twist)], "f64")
    f.load(0, torch.from_numpy(U).cuda())
    print(f"  {dims} defects {f.unitarity(0)}", flush=True)
    f.mc(0.5, 1, n_or, 99)
    got = f.store(0)
    torch.cuda.synchronize()
    d = np.abs(got.cpu().numpy() - a).max()
    print(f"    1 HB + {n_or} OR: max |dU| {d:.3g} (bar {bar:.3g})", flush=True)
    assert bar < 1e-10
    assert d <= bar
