"""Rounding of the SU(N) flow against the same flow in 80-bit arithmetic, all
stage variants.

A stage adds to every link U a term (exp(X) - 1) U that is small (theta =
||X||_F below 0.1 here), so what a good update leaves is the rounding of one
addition: half a unit in the last place of an entry below one, uniform, with
standard deviation 2^-53 / sqrt(12) in each part, independent from stage to
stage.  The small term itself carries the rounding of its products, about
sqrt(N) 2^-53 theta.  Over n stages the root mean square of the links' errors is
therefore below sqrt(2 n (1/12 + N theta^2)) 2^-53.  (An update that accumulates
the products onto U rounds 2 N times per entry and stage at the size of U.)"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import oracle                                      # noqa: E402
from paper_2107_03747_amd import gen, tgf          # noqa: E402

DIMS, EPS, STEPS = (2, 3, 3, 4), 0.01, 16
C, L = np.clongdouble, np.longdouble


def dag(a):
    return np.conj(np.swapaxes(a, -1, -2))


def flow80(U, N, k):
    """Luscher's RK3 of the action's gradient, plane (0, 1) twisted by k; the
    exponential by its series."""
    U = U.astype(C)
    mm = np.matmul
    one = np.eye(N, dtype=C)
    site = np.indices(U.shape[:4])
    corner = (site[3] == 0) & (site[2] == 0)
    phase = np.ones(U.shape[:4], C)
    ang = 8 * np.arctan(L(1)) * k / L(N)
    phase[corner] = np.cos(ang) + 1j * np.sin(ang)

    def shift(a, mu, s):
        return np.roll(a, -s, axis=3 - mu)

    def force(U):
        u = [U[..., m, :, :] for m in range(4)]
        out = []
        for m in range(4):
            S = np.zeros_like(u[0])
            for n in range(4):
                if n == m:
                    continue
                z = phase if (m, n) == (0, 1) else np.conj(phase) if (m, n) == (1, 0) else np.ones_like(phase)
                z = z[..., None, None]
                S += np.conj(z) * mm(mm(shift(u[n], m, 1), dag(shift(u[m], n, 1))), dag(u[n]))
                S += shift(z * mm(mm(dag(shift(u[n], m, 1)), dag(u[m])), u[n]), n, -1)
            W = mm(u[m], S)
            a = (W - dag(W)) / 2
            out.append(np.trace(a, axis1=-2, axis2=-1)[..., None, None] / N * one - a)
        return np.stack(out, axis=4)

    X, theta = np.zeros_like(U), 0.0
    for _ in range(STEPS):
        for a, b in ((L(0), L(1) / 4), (L(-17) / 9, L(8) / 9), (L(-1), L(3) / 4)):
            X = a * X + b * L(EPS) * force(U)
            theta = max(theta, float(np.sqrt((np.abs(X) ** 2).sum((-1, -2))).max()))
            T = np.broadcast_to(one, X.shape)
            for j in range(20, 0, -1):
                T = one + mm(X, T) / L(j)
            U = mm(T, U)
    return U, theta


@pytest.mark.parametrize("N", [2, 3, 4, 5, 6, 7, 8])
def test_rounding_of_the_link_update(N):
    U = gen.near_identity_n(DIMS, N, 0.5, seed=N).numpy()
    tw = (1, 0, 0, 0, 0, 0)
    ref, theta = flow80(U, N, 1)
    far = U.copy()
    oracle.sun_flow(far, DIMS, EPS, STEPS * EPS, 0.0, twist=tw)
    assert np.abs(far - ref.astype(complex)).max() < 1e-14       # the same flow
    bound = np.sqrt(2 * 3 * STEPS * (1 / 12 + N * theta ** 2)) * 2.0 ** -53
    for v in range(tgf.tgf_sun_variant_count(N)):
        f = tgf.Flow([(DIMS, tw)], "f64", nc=N)
        f.set_variant(v)
        f.load(0, torch.from_numpy(U).cuda())
        f.flow(EPS, STEPS * EPS, 0.0)
        got = f.store(0)
        torch.cuda.synchronize()
        d = got.cpu().numpy().astype(C) - ref
        rms = float(np.sqrt((np.abs(d) ** 2).mean()))
        print(f"  SU({N}) variant {v}: rms {rms:.3g}, theta {theta:.3g}, bound {bound:.3g}", flush=True)
        assert rms <= bound
