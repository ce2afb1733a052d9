"""The default stage kernel is chosen per configuration, by its extents and the
storage (lds_by_default in csrc/schedule.h).  A context that holds one box of
either kind launches both kernels: each box gives, bit for bit, the rows and
links of a context of its own, under the kernel that its own default names,
whichever of them ends its flow first, and again when the flow's graph is
replayed."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2107_03747_amd import gen, tgf          # noqa: E402

SMALL, OTHER = (8, 8, 24, 24), (9, 9, 27, 27)
LARGE = {"f64": (9, 9, 306, 306), "f32": (9, 9, 81, 81), "f32c12": (9, 9, 162, 162)}


@pytest.mark.parametrize("storage", ["f64", "f32", "f32c12"])
@pytest.mark.parametrize("longer", ["large", "small"])
def test_default_kernel_of_a_mixed_context(storage, longer):
    names = tgf.variant_names()
    dims = [SMALL, LARGE[storage], OTHER]
    links = [gen.near_identity(d, 0.3, seed=70 + k, device="cuda") for k, d in enumerate(dims)]
    t_end = [0.02, 0.03, 0.02] if longer == "large" else [0.03, 0.02, 0.03]
    want = ["quad_xcd", "site_lds_xcd", "quad_xcd"]
    solo = []
    for k, d in enumerate(dims):
        f = tgf.Flow([d], storage)
        assert names[f.variant] == want[k], d
        f.load(0, links[k])
        rows = f.flow(0.01, t_end[k], 0.01, 2)
        g = tgf.Flow([d], storage)
        g.set_variant(names.index(want[k]))
        g.load(0, links[k])
        assert np.array_equal(g.flow(0.01, t_end[k], 0.01, 2), rows), d
        solo.append((rows, f.store(0)))
    f = tgf.Flow(dims, storage)
    assert names[f.variant] == "quad_xcd"
    for again in range(3):
        print(f"  {storage} {dims} flow {again}", flush=True)
        f.load_all(links)
        rows = f.flow(0.01, t_end, 0.01, 2)
        for k, (r, U) in enumerate(solo):
            assert np.array_equal(rows[: r.shape[0], k], r[:, 0]), dims[k]
            got = f.store(k)
            torch.cuda.synchronize()
            assert torch.equal(got, U), dims[k]
    # one kernel for all, then the default again: the graph follows
    f.set_variant(names.index("quad_xcd"))
    f.load_all(links)
    f.flow(0.01, t_end, 0.01, 2)
    assert torch.equal(f.store(0), solo[0][1])
    f.set_variant(-1)
    f.load_all(links)
    f.flow(0.01, t_end, 0.01, 2)
    assert torch.equal(f.store(1), solo[1][1])
