"""The quad stage kernel (one wave per direction and 64-site tile) where its
paths differ: tiles closed under the shift in direction 0 and 1, in 0 only, in
neither, tiles with idle lanes, extents of 2, every plane twisted -- one RK3
step against the FP64 oracle, links entry by entry, and a batch of all of them
bitwise equal to each box alone.

Tolerance: a stage sums eighteen loops of three products of 3-term rows and
adds an exponential's product of 3 terms to a link entry of size at most 1; the
rounding of a step of three stages stays below 3 x (18 x 3 x 3 eps + 3 + 3)
units of 2^-53 (FP64), and below twelve units of 2^-24 per stage (FP32: the
force enters times eps = 0.02, so only the storage of the link, the product
with its first-order increment and the input's rounding count in full)."""

import numpy as np
import pytest
import torch

import oracle
from paper_2107_03747_amd import gen, tgf

pytestmark = pytest.mark.gpu

DIMS = [(8, 8, 3, 2), (16, 4, 3, 3), (4, 4, 5, 3), (32, 2, 3, 2), (64, 2, 2, 2), (2, 32, 3, 2),
        (10, 10, 3, 2), (3, 5, 4, 7), (2, 2, 2, 2), (2, 2, 2, 3), (65, 3, 2, 2), (9, 7, 2, 2)]
TWIST = (1, 2, 1, 2, 1, 2)
EPS = 0.02
TOL = {"f64": 3 * (18 * 3 * 3 * EPS + 6) * 2.0 ** -52, "f32": 36 * 2.0 ** -24,
       "f32c12": 36 * 2.0 ** -24}


@pytest.mark.parametrize("storage", ["f64", "f32", "f32c12"])
def test_quad_paths(storage):
    v = tgf.variant_names().index("quad_xcd")
    Us = [gen.near_identity(d, 0.35, seed=90 + k).numpy().copy() for k, d in enumerate(DIMS)]
    dev = [torch.from_numpy(U).cuda() for U in Us]
    f = tgf.Flow([(d, TWIST) for d in DIMS], storage)
    f.set_variant(v)
    f.load_all(dev)
    rows = f.flow(EPS, EPS, 0.0)
    for k, d in enumerate(DIMS):
        ref = Us[k].copy()
        oracle.rk3_step(ref, d, EPS, twist=TWIST)
        got = f.store(k)
        torch.cuda.synchronize()
        e = np.abs(got.cpu().numpy() - ref).max()
        print(f"  {storage} {d}: max |dU| {e:.3g} (tol {TOL[storage]:.3g})", flush=True)
        assert e <= TOL[storage]
        g = tgf.Flow([(d, TWIST)], storage)
        g.set_variant(v)
        g.load(0, dev[k])
        solo = g.flow(EPS, EPS, 0.0)
        assert np.array_equal(solo[:, 0], rows[:, k]), d
        assert torch.equal(g.store(0), got), d
