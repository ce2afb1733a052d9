"""SU(N) kernels at the edges of their paths: one RK3 step of every stage
variant against the FP64 oracle, links entry by entry.

* The exponential's branches: step sizes whose X spans the polynomial degrees
  (theta = ||X||_F up to 0.059, 0.21, 0.49, 0.88, 1.4) and the halved-argument
  branch above, the closed form of N = 2 and the Cayley-Hamilton series of
  N = 3 included.
* Boxes whose sites fill no group evenly (81, 24 and 54 sites: groups hold 64/N
  or 4 or 1 sites), extents of 2 (n + mu and n - mu the same site), and every
  plane twisted.

Tolerance: one step is three stages; each forms links of unit entries by sums
of at most 13 products of N terms and an exponential whose rounding grows with
theta (products of matrices of norm up to e^theta, and one doubling of the
error per squaring), so 3 x 13 x N x 2^-52 (1 + theta) (1 + 2 theta) bounds it
with room for the oracle's own rounding.
"""

import numpy as np
import pytest
import torch

import oracle
from paper_2107_03747_amd import gen, tgf

pytestmark = pytest.mark.gpu


def one_step_all_variants(N, dims, twist, eps, start=0.5):
    U = gen.near_identity_n(dims, N, start, seed=7 + N).numpy().copy()
    F = oracle.sun_force(U, dims, twist=twist)
    theta = float(np.sqrt((np.abs(F) ** 2).sum((-1, -2))).max()) * eps   # X <= eps |F| in size
    ref = U.copy()
    oracle.sun_rk3_step(ref, dims, eps, twist=twist)
    tol = 3 * 13 * N * 2.0 ** -52 * (1 + theta) * (1 + 2 * theta)
    for v in range(tgf.tgf_sun_variant_count(N)):
        f = tgf.Flow([(dims, twist)], "f64", nc=N)
        f.set_variant(v)
        f.load(0, torch.from_numpy(U).cuda())
        f.flow(eps, eps, 0.0)
        got = f.store(0)
        torch.cuda.synchronize()
        d = np.abs(got.cpu().numpy() - ref).max()
        print(f"  SU({N}) {dims} eps {eps} theta <= {theta:.3g} variant {v}: max |dU| {d:.3g} "
              f"(tol {tol:.3g})", flush=True)
        assert d <= tol


@pytest.mark.parametrize("eps", [0.002, 0.03, 0.1, 0.25, 1.0])
@pytest.mark.parametrize("N", [2, 3, 4, 5, 6, 7, 8])
def test_exponential_branches(N, eps):
    one_step_all_variants(N, (2, 2, 2, 3), (1, 0, 0, 0, 0, 0), eps)


@pytest.mark.parametrize("dims", [(3, 3, 3, 3), (2, 3, 3, 3)])
@pytest.mark.parametrize("N", [2, 3, 4, 5, 6, 7, 8])
def test_ragged_groups_all_planes_twisted(N, dims):
    one_step_all_variants(N, dims, (1, N - 1, 1, N // 2, 1, N - 1), 0.02)


@pytest.mark.parametrize("dims", [(3, 3, 3, 3), (2, 3, 3, 5)])
@pytest.mark.parametrize("N", [2, 3, 4, 5, 6, 7, 8])
def test_measurement_of_ragged_tiles_all_planes_twisted(N, dims):
    """Rows of every variant's measurement on boxes of two part-filled tiles
    (81 and 90 sites; work-groups own a plane pair, or a part of the sites).
    An entry of a leaf is off by at most 2 (3 N) ulps, so is one of G; the
    density sums 6 N^2 products of two such entries of size below one."""
    tw = (1, N - 1, 1, N // 2, 1, N - 1)
    U = gen.near_identity_n(dims, N, 0.5, seed=31 + N).numpy().copy()
    ref = oracle.sun_measure(U, dims, twist=tw)
    V = int(np.prod(dims))
    ulp = 6 * N * 2.0 ** -52
    tol = {1: 12 * N * N * ulp, 3: ulp, 4: V * 6 * N * N * ulp, 5: 6 * N * V * ulp}
    for v in range(tgf.tgf_sun_variant_count(N)):
        f = tgf.Flow([(dims, tw)], "f64", nc=N)
        f.set_variant(v)
        f.load(0, torch.from_numpy(U).cuda())
        row = np.asarray(f.measure())[0]
        for col, key in ((1, "E"), (3, "plaq"), (4, "Q"), (5, "action")):
            d = abs(float(row[col]) - float(ref[key]))
            print(f"  SU({N}) {dims} variant {v} {key}: off {d:.3g} (tol {tol[col]:.3g})", flush=True)
            assert d <= tol[col]
