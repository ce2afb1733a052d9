"""The default stage kernel on boxes whose tiles run in columns (an n3 slice of
more than 128 tiles: columns of four (n0, n1) planes, 16, 64, 36 and 25 tiles
wide here): links entry by entry against the oracle after two steps, within the
bars of the other column order's test, and the same box in a batch with a
site-order box bitwise its solo links."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import oracle                                      # noqa: E402
from paper_2107_03747_amd import gen, tgf          # noqa: E402

OTHER = (8, 8, 24, 24)


@pytest.mark.parametrize("storage", ["f64", "f32", "f32c12"])
@pytest.mark.parametrize("dims", [(16, 16, 72, 4), (32, 32, 16, 5), (24, 24, 24, 4), (20, 20, 60, 3)])
def test_links_in_tile_columns(dims, storage):
    v = tgf.variant_names().index("quad_xcd")
    U = gen.near_identity(dims, 0.3, seed=91).numpy().copy()
    W = gen.near_identity(OTHER, 0.3, seed=92).numpy().copy()
    ref = U.copy()
    oracle.flow(ref, dims, 0.01, 0.02, 0.0)
    out = []
    for batch in ([dims], [OTHER, dims]):
        f = tgf.Flow(batch, storage)
        f.set_variant(v)
        f.load_all([torch.from_numpy(U if d == dims else W).cuda() for d in batch])
        f.flow(0.01, 0.02, 0.0)
        out.append(f.store(len(batch) - 1))
        torch.cuda.synchronize()
    d = np.abs(out[0].cpu().numpy() - ref).max()
    print(f"  tile columns {dims} {storage}: max |dU| {d:.3g}", flush=True)
    assert d <= (1e-13 if storage == "f64" else 3e-6)      # two steps
    assert torch.equal(out[0], out[1])
