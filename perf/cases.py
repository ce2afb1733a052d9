"""The work that a user of this framework has it do, as cases that can be timed.

Every case is a batch of boxes worked on through ``tgf.Flow`` (and, for the
measurement without a context, the C entry point of the same module):

* ``flow``  load the links, flow them (RK3, rows of t, E, t2E, plaquette, Q,
            action along the way), write the flowed links back;
* ``mc``    load the links, hybrid over-relaxation sweeps, write them back;
* ``obs``   load the links, measure them (rows, slice charges, per-site
            densities, and the measurement without a context), write them back.

``exact`` is the same in plain torch, 64 bits.  A flow in a 32-bit storage
carries 32-bit accuracy in all it returns, so its rows and links are handed on
in 32 bits, as a program that keeps such results would hold them.
"""

from __future__ import annotations

import math

import numpy as np
import torch

EPS = 0.01
PAPER_TWIST = "1,0,0,0,0,0"
DEV = "cuda"


# ---------------------------------------------------------------------------
# cases

def _case(name, kind, boxes, **kw):
    c = {"name": name, "kind": kind, "boxes": boxes, "storage": "f64", "nc": 0,
         "twist": PAPER_TWIST, "start": "near", "steps": 0, "meas_dt": 0.1, "reunit": 0,
         "n_hybrid": 0, "n_or": 0, "b": 0.0}
    c.update(kw)
    return c


def listed():
    return [
        # the benchmark's ensemble: 96 configurations of L = 6, 8, 10 flowed to
        # sqrt(8t) = 0.3 L, measured every 0.1, reunitarised every 10 steps
        _case("flow_ensemble_f32c12", "flow", "8x8x24x24*64,6x6x18x18*16,10x10x30x30*16",
              storage="f32c12", reunit=10),
        # one small box on its own: the latency of a flow, rows close together
        _case("flow_single_f32c12", "flow", "4x4x12x12*1", storage="f32c12", steps=32,
              meas_dt=0.04, reunit=10),
        # odd extents, which fill no wavefront and no work-group evenly
        _case("flow_odd_f32c12", "flow", "5x5x15x15*6,7x7x21x21*6,9x9x27x27*2",
              storage="f32c12", steps=40, reunit=10),
        # a hot start on the paper's largest lattice, full 32-bit storage
        _case("flow_hot16_f32", "flow", "16x16x48x48*1", storage="f32", start="hot", steps=24,
              reunit=10),
        # the first steps of the large box (many times any cache)
        _case("flow_large_f32c12", "flow", "32x32x96x96*1", storage="f32c12", start="hot",
              steps=6),
        # a mixed ensemble in 64 bits
        _case("flow_ensemble_f64", "flow", "8x8x24x24*24,6x6x18x18*8,12x12x36x36*2", steps=30),
        # one mid-size box in 64 bits to sqrt(8t) = 0.3 L
        _case("flow_single_f64", "flow", "6x6x18x18*1"),
        # generation: one hybrid sweep (heat bath + over-relaxation) of an ensemble
        _case("mc_ensemble", "mc", "8x8x24x24*32,6x6x18x18*8,10x10x30x30*8", n_hybrid=1, n_or=8,
              b=0.5),
        # measurements on flowed-size lattices: rows, slice charges, densities
        _case("obs_f64", "obs", "16x16x48x48*2"),
        # SU(4): an ensemble of small boxes of the l^2 x (N l)^2 geometry
        _case("flow_su4", "flow", "4x4x16x16*48", nc=4, steps=10),
        # SU(8), the largest group
        _case("flow_su8", "flow", "4x4x32x32*4", nc=8, steps=4),
        # SU(5) on one odd box with another twist: few sites, latency again
        _case("flow_su5_odd", "flow", "3x3x15x15*1", nc=5, steps=16, twist="2,0,0,0,0,0",
              meas_dt=0.04),
    ]


def _boxes(text):
    out = []
    for part in text.split(","):
        d, n = part.split("*")
        out += [tuple(int(x) for x in d.split("x"))] * int(n)
    return out


def _draw_box(rng, nc, even, vmax):
    """A box of at most vmax sites: mostly l x l x Nl x Nl, now and then any extents."""
    while True:
        if rng.random() < 0.75:
            lo, hi = (2, 6) if nc else (3, 16)
            l = rng.randint(lo, hi)
            l += (l & 1) if even else 0
            d = (l, l, (nc or 3) * l, (nc or 3) * l)
        else:
            d = tuple(int(round(math.exp(rng.uniform(math.log(2), math.log(24)))))
                      for _ in range(4))
            d = tuple(x + (x & 1) for x in d) if even else d
        if 500 <= math.prod(d) <= vmax:
            return d


def draw(rng):
    """One more case: kind, storage, group, boxes (a batch of one or two
    extents), start, twist and schedule over the ranges of the listed ones."""
    kind = rng.choice(("flow",) * 7 + ("mc",) * 2 + ("obs",))
    nc = rng.choice((2, 3, 4, 5, 6, 7, 8)) if kind == "flow" and rng.random() < 0.35 else 0
    storage = "f64" if nc or kind == "mc" else rng.choice(("f32c12", "f32c12", "f32", "f64"))
    # sites x (relative cost of one) stays below the largest listed case's
    cost = {"f32c12": 1.0, "f32": 1.3, "f64": 3.0}[storage] * ((nc / 3) ** 3 * 1.5 if nc else 1.0)
    vmax = max(2000, int(2.4e6 / cost))
    total = int(math.exp(rng.uniform(math.log(1500), math.log(vmax))))
    parts = []
    for _ in range(rng.choice((1, 1, 2))):
        d = _draw_box(rng, nc, kind == "mc", max(total, 1500))
        parts.append("x".join(map(str, d)) + "*%d" % max(1, min(64, total // (2 * math.prod(d)))))
    top = nc or 3
    twist = PAPER_TWIST if rng.random() < 0.6 else ",".join(str(rng.randrange(top)) for _ in range(6))
    c = _case("", kind, ",".join(parts), storage=storage, nc=nc, twist=twist,
              start="near" if nc else rng.choice(("near", "near", "hot")),
              meas_dt=rng.choice((0.02, 0.05, 0.1)))
    del c["name"]
    if kind == "flow":
        c["steps"] = rng.randint(3, 6) if nc > 5 else rng.randint(4, 30)
        c["reunit"] = rng.choice((0, 5, 10)) if storage != "f64" else 0
    elif kind == "mc":
        c["n_hybrid"], c["n_or"], c["b"] = rng.randint(1, 2), rng.randint(0, 6), rng.uniform(0.33, 1.2)
    return c


# ---------------------------------------------------------------------------
# inputs

def _twist(case):
    return tuple(int(x) for x in case["twist"].split(","))


def _t_end(case, d):
    return case["steps"] * EPS if case["steps"] else 0.09 * d[0] * d[0] / 8


def _links(d, N, start, seed):
    """Links [d3, d2, d1, d0, 4, N, N]: exp(i e H) with Gaussian H (e 0.2, 0.3
    or 0.4 in turn), or Haar-distributed SU(3)."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    n = 4 * math.prod(d)
    if start == "hot":
        z = torch.view_as_complex(torch.randn(n, 2, 3, 2, dtype=torch.float64, device=DEV, generator=g))
        a = z[:, 0] / torch.linalg.vector_norm(z[:, 0], dim=-1, keepdim=True)
        b = z[:, 1] - (a.conj() * z[:, 1]).sum(-1, keepdim=True) * a
        b = b / torch.linalg.vector_norm(b, dim=-1, keepdim=True)
        r = torch.stack([a[:, 1] * b[:, 2] - a[:, 2] * b[:, 1], a[:, 2] * b[:, 0] - a[:, 0] * b[:, 2],
                         a[:, 0] * b[:, 1] - a[:, 1] * b[:, 0]], dim=-1).conj()
        U = torch.stack([a, b, r], dim=1)
    else:
        z = torch.view_as_complex(torch.randn(n, N, N, 2, dtype=torch.float64, device=DEV, generator=g))
        X = (0.5 * math.sqrt(0.5)) * (z - z.mH)          # anti-Hermitian
        X = X - (torch.diagonal(X, dim1=-2, dim2=-1).sum(-1) / N)[:, None, None] * torch.eye(
            N, dtype=torch.complex128, device=DEV)
        X = X * (0.2, 0.3, 0.4)[seed % 3]
        # scaled so that the Taylor polynomial of degree 14 is exact to rounding
        U = _exp(X / 16, 14)
        for _ in range(4):
            U = _mm(U, U)
    return U.reshape(d[3], d[2], d[1], d[0], 4, N, N).contiguous()


def _inputs(case, seed):
    N = case["nc"] or 3
    return [_links(d, N, case["start"], 1000 * seed + k) for k, d in enumerate(_boxes(case["boxes"]))]


def prepare(case, seed):
    from paper_2107_03747_amd import tgf
    boxes, tw = _boxes(case["boxes"]), _twist(case)
    f = tgf.Flow([(d, tw) for d in boxes], case["storage"], nc=case["nc"] or None)
    links = _inputs(case, seed)
    # where the links go afterwards: one buffer for the whole batch
    flat = torch.empty(sum(u.numel() for u in links), dtype=torch.complex128, device=DEV)
    back, o = [], 0
    for u in links:
        back.append(flat[o:o + u.numel()].view(u.shape))
        o += u.numel()
    s = {"case": case, "seed": seed, "tgf": tgf, "f": f, "links": links, "flat": flat, "back": back,
         "t_end": [_t_end(case, d) for d in boxes]}
    if case["kind"] == "obs":
        s["geoms"] = [tgf.make_geoms([(d, tw)]) for d in boxes]
        s["obs"] = torch.empty(len(boxes), 6, dtype=torch.float64, device=DEV)
    torch.cuda.synchronize()
    return s


def run(s):
    case, f = s["case"], s["f"]
    f.load_all(s["links"])
    out = {}
    if case["kind"] == "flow":
        out["rows"] = f.flow(EPS, s["t_end"], case["meas_dt"], case["reunit"])
    elif case["kind"] == "mc":
        f.mc(case["b"], case["n_hybrid"], case["n_or"], seed=s["seed"])
    else:
        tgf = s["tgf"]
        out["rows"] = f.measure()
        out["slices"] = f.slice_charge(3)
        d = [f.densities(k) for k in range(f.n)]
        out["e"], out["q"] = torch.cat([x[0] for x in d]), torch.cat([x[1] for x in d])
        stream = torch.cuda.current_stream().cuda_stream
        for k in range(f.n):
            tgf.check(tgf.tgf_measure_noalloc(s["geoms"][k], s["links"][k].data_ptr(), 0.5,
                                              s["obs"][k].data_ptr(), stream))
        out["obs"] = s["obs"]
    for k, u in enumerate(s["back"]):
        f.store(k, out=u)
    out["links"] = s["flat"]
    if case["storage"] != "f64":
        out = {k: v.astype(np.float32) if isinstance(v, np.ndarray) else
               v.to(torch.complex64 if v.is_complex() else torch.float32) for k, v in out.items()}
    return out


def work(case):
    """Bytes and operations of one pass.  A flow: the canonical links read and
    written once, and per step and site the links read and written and the
    accumulator written, updated and read once in each of the three stages (a
    stage needs every link of the one before).  Monte Carlo: per link update
    the links read by its launch, and the link written."""
    boxes, N = _boxes(case["boxes"]), case["nc"] or 3
    nn, rb = N * N, 8 if case["storage"] == "f64" else 4
    by = fl = 0.0
    for d in boxes:
        V = math.prod(d)
        by += 2 * V * 4 * nn * 16
        if case["kind"] == "flow":
            steps = len(_steps(0.0, _t_end(case, d)))
            entries = 6 if case["storage"] == "f32c12" else nn
            x = nn if case["nc"] else 4
            by += V * steps * 2 * rb * (3 * 2 * 4 * entries + 4 * 4 * x)
            # 18 closed loops of three products, four exponentials and updates
            fl += V * steps * 3 * ((18 * 2 * 132 + 18 * 70 + 4 * 490) if not case["nc"] else
                                   (4 * 19 * 8 * N ** 3 + 4 * 64 * nn))
        elif case["kind"] == "mc":
            n = case["n_hybrid"] * (1 + case["n_or"]) * 4 * V
            by += n * 1296.0
            fl += n * 3402.0
        else:
            by += 4 * V * 4 * nn * 2 * rb + 16 * V
            fl += 4 * V * 6 * (4 * 3 * 132 + 100)
    return {"bytes": by, "flops": fl}


# ---------------------------------------------------------------------------
# the same in plain torch, 64 bits

def _mm(a, b):
    if a.shape[-1] > 3:
        return torch.matmul(a, b)
    return (a.unsqueeze(-1) * b.unsqueeze(-3)).sum(-2)


def _dag(a):
    return a.conj().transpose(-1, -2).resolve_conj().contiguous()


def _exp(X, degree=12):
    E = torch.eye(X.shape[-1], dtype=X.dtype, device=X.device)
    T = E + X / degree
    for k in range(degree - 1, 0, -1):
        T = E + _mm(T, X) / k
    return T


class _Lattice:
    """Boxes of one extent, U[mu] of shape [n, d3, d2, d1, d0, N, N]."""

    def __init__(self, d, tw, N):
        self.d, self.N, self.Z = d, N, {}
        planes = [(m, n) for m in range(4) for n in range(m + 1, 4)]
        x = torch.meshgrid(*[torch.arange(d[m], device=DEV) for m in (3, 2, 1, 0)], indexing="ij")[::-1]
        for (m, n), k in zip(planes, tw):
            z = torch.ones(x[0].shape, dtype=torch.complex128, device=DEV)
            z[(x[m] == 0) & (x[n] == 0)] = complex(math.cos(2 * math.pi * k / N),
                                                   math.sin(2 * math.pi * k / N))
            self.Z[m, n] = z[None, ..., None, None]
        self.planes = planes
        self.parity = (x[0] + x[1] + x[2] + x[3]) % 2
        self.site = x[0] + d[0] * (x[1] + d[1] * (x[2] + d[2] * x[3]))

    @staticmethod
    def up(a, m):
        return torch.roll(a, -1, 4 - m)

    @staticmethod
    def dn(a, m):
        return torch.roll(a, 1, 4 - m)

    def omega(self, U):
        """U_mu(n) times the twisted staple sum, for every mu."""
        om = [torch.zeros_like(u) for u in U]
        S = [torch.zeros_like(u) for u in U]
        for m, n in self.planes:
            Z = self.Z[m, n]
            A = _mm(U[m], self.up(U[n], m))
            B = _mm(U[n], self.up(U[m], n))
            P = Z.conj() * _mm(A, _dag(B))
            om[m] += P
            om[n] += _dag(P)
            S[m] += self.dn(Z * _mm(_dag(A), U[n]), n)
            S[n] += self.dn(Z.conj() * _mm(_dag(B), U[m]), m)
        return [o + _mm(u, s) for o, u, s in zip(om, U, S)]

    def step(self, U, eps):
        X = [torch.zeros_like(u) for u in U]
        eye = torch.eye(self.N, dtype=torch.complex128, device=DEV) / self.N
        for a, b in ((0.0, 0.25), (-17 / 9, 8 / 9), (-1.0, 0.75)):
            om = self.omega(U)
            for m in range(4):
                A = 0.5 * (om[m] - _dag(om[m]))
                A = A - torch.diagonal(A, dim1=-2, dim2=-1).sum(-1)[..., None, None] * eye
                X[m] = a * X[m] - (b * eps) * A
                U[m] = _mm(_exp(X[m]), U[m])
        return U

    def measure(self, U):
        """e(n), q(n), and the sums over the planes of Re Tr Z* P (per site)."""
        G, p = {}, 0
        for m, n in self.planes:
            P = self.Z[m, n].conj() * _mm(_mm(U[m], self.up(U[n], m)), _dag(_mm(U[n], self.up(U[m], n))))
            p = p + torch.diagonal(P, dim1=-2, dim2=-1).sum(-1).real
            C = P + self.dn(_mm(_dag(U[n]), _mm(P, U[n])), n)
            C = C + self.dn(_mm(_dag(U[m]), _mm(C, U[m])), m)
            G[m, n] = -0.125j * (C - _dag(C))
        tr = lambda a, b: (a * b.conj()).real.sum((-1, -2))  # noqa: E731
        e = sum(tr(g, g) for g in G.values())
        q = (tr(G[0, 1], G[2, 3]) - tr(G[0, 2], G[1, 3]) + tr(G[0, 3], G[1, 2])) / (4 * math.pi ** 2)
        return e, q, p

    def rows(self, U, t):
        """[n, 6]: t, E, t2E, plaquette, Q, action."""
        e, q, p = self.measure(U)
        V = math.prod(self.d)
        s = lambda v: v.reshape(v.shape[0], -1).sum(1)  # noqa: E731
        E, pl = s(e) / V, s(p)
        return torch.stack([torch.full_like(E, t), E, t * t * E, pl / (6 * self.N * V), s(q),
                            6.0 * self.N * V - pl], 1).cpu().numpy()


def _steps(t0, t_end):
    n = 0
    while t0 + (n + 1) * EPS <= t_end + 1e-12:
        n += 1
    rest = t_end - (t0 + n * EPS)
    return [EPS] * n + ([rest] if rest > 1e-12 else [])


def _on_grid(t, dt):
    return dt > 0 and abs(t - math.floor(t / dt + 0.5) * dt) <= 1e-9


def _philox(ctr, k0, k1):
    """Philox4x32-10 on int64 tensors that hold 32-bit words."""
    M = 0xFFFFFFFF
    hi = lambda a, b: (((b >> 16) * a) + (((b & 0xFFFF) * a) >> 16)) >> 16  # noqa: E731
    x, y, z, w = ctr
    for _ in range(10):
        h0, l0 = hi(0xD2511F53, x), (0xD2511F53 * x) & M
        h1, l1 = hi(0xCD9E8D57, z), (0xCD9E8D57 * z) & M
        x, y, z, w = (h1 ^ y ^ k0) & M, l1, (h0 ^ w ^ k1) & M, l0
        k0, k1 = (k0 + 0x9E3779B9) & M, (k1 + 0xBB67AE85) & M
    return x, y, z, w


def _unit(x):
    return (x.double() + 0.5) / 4294967296.0


def _su2_draw(alpha, site, sweep, z, cfg, key):
    """Unit quaternions with y0 ~ sqrt(1 - y0^2) exp(alpha y0)."""
    y0 = torch.ones_like(alpha)
    todo = torch.ones_like(alpha, dtype=torch.bool)
    sw = torch.full_like(site, sweep)
    for att in range(256):
        if not bool(todo.any()):
            break
        u1, u2, u3, u4 = (_unit(v) for v in _philox((site, sw, torch.full_like(site, z | att), cfg), *key))
        ex = torch.exp(-2 * alpha)
        creutz = 1 + torch.log(u1 * (1 - ex) + ex) / alpha
        lam2 = -(torch.log(u1) + torch.cos(2 * math.pi * u2) ** 2 * torch.log(u3)) / (2 * alpha)
        y = torch.where(alpha < 1e-8, 2 * u1 - 1, torch.where(alpha < 2, creutz, 1 - 2 * lam2))
        ok = torch.where(alpha < 2, u2 * u2 <= 1 - y * y, u4 * u4 <= 1 - lam2) & todo
        y0 = torch.where(ok, y, y0)
        todo = todo & ~ok
    r = _philox((site, sw, torch.full_like(site, z | 0xFFFF), cfg), *key)
    ct, ph = 2 * _unit(r[0]) - 1, 2 * math.pi * _unit(r[1])
    st, rad = torch.sqrt((1 - ct * ct).clamp(min=0)), torch.sqrt((1 - y0 * y0).clamp(min=0))
    y = torch.stack([y0, rad * st * torch.cos(ph), rad * st * torch.sin(ph), rad * ct], -1)
    y[todo] = torch.tensor([1.0, 0, 0, 0], dtype=torch.float64, device=DEV)
    return y


def _block(q):
    q0, q1, q2, q3 = q.unbind(-1)
    return torch.stack([torch.stack([torch.complex(q0, q3), torch.complex(q2, q1)], -1),
                        torch.stack([torch.complex(-q2, q1), torch.complex(q0, -q3)], -1)], -2)


def _mc(L, U, cfgs, case, seed):
    key, sweep = (seed & 0xFFFFFFFF, seed >> 32), 0
    cfg_all = torch.tensor(cfgs, device=DEV).view(-1, 1, 1, 1, 1).expand(U[0].shape[:5])
    for _ in range(case["n_hybrid"]):
        for o in range(case["n_or"] + 1):
            for mu in range(4):
                for par in (0, 1):
                    sel = (L.parity == par)[None].expand(U[0].shape[:5])
                    S = 0
                    for nu in range(4):
                        if nu == mu:
                            continue
                        Z = L.Z[mu, nu] if mu < nu else L.Z[nu, mu].conj()
                        A = _mm(U[mu], L.up(U[nu], mu))
                        S = S + Z.conj() * _mm(L.up(U[nu], mu), _dag(_mm(U[nu], L.up(U[mu], nu))))
                        S = S + L.dn(Z * _mm(_dag(A), U[nu]), nu)
                    u, om = U[mu][sel], _mm(U[mu][sel], S[sel])
                    site, cfg = L.site[None].expand(sel.shape)[sel], cfg_all[sel]
                    for sub, (a, b) in enumerate(((0, 1), (0, 2), (1, 2))):
                        c = torch.stack([om[:, a, a].real + om[:, b, b].real,
                                         -(om[:, a, b].imag + om[:, b, a].imag),
                                         om[:, b, a].real - om[:, a, b].real,
                                         om[:, b, b].imag - om[:, a, a].imag], -1)
                        k = torch.linalg.vector_norm(c, dim=-1)
                        C = _block(c / k[:, None])
                        A = C
                        if o == 0:
                            y = _su2_draw(18 * case["b"] * k / 3, site, sweep, (mu << 24) | (sub << 16),
                                          cfg, key)
                            A = _block(y)
                        A = (A.unsqueeze(-1) * C.unsqueeze(-3)).sum(-2)
                        u, om = u.clone(), om.clone()
                        for m in (u, om):
                            m[:, (a, b)] = (A.unsqueeze(-1) * m[:, (a, b)].unsqueeze(-3)).sum(-2)
                    U[mu][sel] = u
            sweep += 1
    return U


def exact(case, seed):
    boxes, N, tw = _boxes(case["boxes"]), case["nc"] or 3, _twist(case)
    if case["kind"] == "flow":
        # about 80 N x N products per site and stage
        cost = sum(math.prod(d) * len(_steps(0.0, _t_end(case, d))) for d in boxes)
        if cost * (N / 3) ** 3 > 1.2e8:
            return None
    links = _inputs(case, seed)
    back = [None] * len(boxes)
    meas = [None] * len(boxes)      # rows of each configuration
    dens, slices = [None] * len(boxes), [None] * len(boxes)
    for d in dict.fromkeys(boxes):
        ks = [k for k, x in enumerate(boxes) if x == d]
        W = torch.stack([links[k] for k in ks])
        U = [W[..., m, :, :].contiguous() for m in range(4)]
        del W
        L = _Lattice(d, tw, N)
        rows = []
        if case["kind"] == "flow":
            t, t_end = 0.0, _t_end(case, d)
            st = _steps(0.0, t_end)
            if _on_grid(0.0, case["meas_dt"]) or not st:
                rows.append(L.rows(U, 0.0))
            for k, eps in enumerate(st):
                U = L.step(U, eps)
                t = t_end if (k == len(st) - 1 and eps != EPS) else (k + 1) * EPS
                if _on_grid(t, case["meas_dt"]) or k == len(st) - 1:
                    rows.append(L.rows(U, t))
        elif case["kind"] == "mc":
            U = _mc(L, U, ks, case, seed)
        else:
            rows.append(L.rows(U, 0.0))
            e, q, _ = L.measure(U)
            for j, k in enumerate(ks):
                dens[k] = (e[j].reshape(-1), q[j].reshape(-1))
                slices[k] = q[j].sum((1, 2, 3)).cpu().numpy()
        for j, k in enumerate(ks):
            meas[k] = [r[j] for r in rows]
            back[k] = torch.stack([u[j] for u in U], -3).reshape(-1)
        del U
    out = {"links": torch.cat(back)}
    if case["kind"] == "flow":
        n = max(len(m) for m in meas)
        out["rows"] = np.stack([np.stack([m[min(r, len(m) - 1)] for m in meas]) for r in range(n)])
    elif case["kind"] == "obs":
        out["rows"] = np.stack([m[0] for m in meas])
        out["slices"] = np.zeros((len(boxes), max(d[3] for d in boxes)))
        for k, v in enumerate(slices):
            out["slices"][k, :len(v)] = v
        out["e"], out["q"] = (torch.cat([x[j] for x in dens]) for j in (0, 1))
        obs = out["rows"].copy()
        obs[:, 0] = 0.5
        obs[:, 2] = 0.25 * obs[:, 1]
        out["obs"] = obs
    return out
