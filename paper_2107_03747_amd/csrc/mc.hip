// mc.hip -- Monte Carlo generation of twisted SU(3) gauge fields for gfx950.
//
// Method (arXiv 2107.03747, sec. 3.1): configurations of the twisted Wilson
// action S_W = 3b sum_n sum_{mu != nu} Tr[1 - Z^*_{mu nu}(n) P_{mu nu}(n)]
// are generated by hybrid over-relaxation: one heat-bath sweep followed by
// over-relaxation sweeps.  With beta = 18 b the part of S_W that depends on
// one link is -(beta/3) Re Tr[Omega], Omega = U_mu(n) S the twisted staple
// sum (the same Omega whose projection is the flow force).
//
// A link is updated in the three SU(2) subgroups on rows (0,1), (0,2), (1,2)
// in turn (Cabibbo-Marinari): U -> A U with A in the subgroup.  For the 2x2
// block w of Omega on rows (a, b), Re Tr[A Omega] - const = x . c with x the
// unit quaternion of A = [[x0 + i x3, x2 + i x1], [-x2 + i x1, x0 - i x3]] and
//   c = (Re w_aa + Re w_bb, -(Im w_ab + Im w_ba), Re w_ba - Re w_ab, Im w_bb - Im w_aa).
// With C the SU(2) element of c/|c|:
//   heat bath        A = Y C, Y drawn with density ~ exp(alpha y0) on SU(2),
//                    alpha = beta |c| / 3 (Creutz's method for alpha < 2,
//                    Kennedy-Pendleton's otherwise, at most 256 attempts);
//   over-relaxation  A = C C, which keeps Re Tr[Omega].
// A sweep visits mu = 0..3 and, for each, the even then the odd sites
// (n0+n1+n2+n3 even / odd): the links of one direction and parity have no
// staple in common with each other, so each such set is one launch and is
// updated in place.
//
// Random numbers: Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11) keyed by
// the 64-bit seed, counter (site, sweep, mu << 24 | subgroup << 16 | attempt,
// configuration), attempt 0xFFFF for the direction of (y1, y2, y3); a 32-bit
// output x becomes the double (x + 1/2) 2^-32.  The counter names every draw,
// so a chain does not depend on the launch shape, the batch composition or
// the order of configurations.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "launch.h"
#include "lattice_dev.h"
#include "layout.h"
#include "su3_dev.h"

namespace tgf {

struct Ctr {
    uint32_t x, y, z, w;
};

// Philox4x32-10: ten rounds of two 32x32 -> 64-bit products (multipliers
// 0xD2511F53, 0xCD9E8D57) with the key advanced by the Weyl increments
// (0x9E3779B9, 0xBB67AE85) after every round.
__device__ __forceinline__ Ctr philox4x32_10(Ctr c, uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; r++) {
        const uint32_t hi0 = __umulhi(0xD2511F53u, c.x), lo0 = 0xD2511F53u * c.x;
        const uint32_t hi1 = __umulhi(0xCD9E8D57u, c.z), lo1 = 0xCD9E8D57u * c.z;
        c = Ctr{hi1 ^ c.y ^ k0, lo1, hi0 ^ c.w ^ k1, lo0};
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c;
}

__device__ __forceinline__ double unit_open(uint32_t x) {
    return ((double)x + 0.5) * (1.0 / 4294967296.0);
}

constexpr double kTwoPi = 6.28318530717958647692;

// Unit quaternion y with y0 ~ sqrt(1 - y0^2) exp(alpha y0) and (y1, y2, y3)
// uniform on the sphere of radius sqrt(1 - y0^2).
__device__ void su2_heatbath_draw(double alpha, Ctr ctr, uint32_t k0, uint32_t k1, double y[4]) {
    double y0 = 1.0;
    bool ok = false;
    for (uint32_t att = 0; att < 256u && !ok; att++) {
        Ctr q = ctr;
        q.z |= att;
        const Ctr r = philox4x32_10(q, k0, k1);
        const double u1 = unit_open(r.x), u2 = unit_open(r.y), u3 = unit_open(r.z),
                     u4 = unit_open(r.w);
        if (alpha < 1e-8) {
            // no preferred direction: y0 with the bare Haar weight
            y0 = 2.0 * u1 - 1.0;
            ok = u2 * u2 <= 1.0 - y0 * y0;
        } else if (alpha < 2.0) {
            // Creutz: y0 from exp(alpha y0) by inversion, accept with sqrt(1 - y0^2)
            const double e = exp(-2.0 * alpha);
            y0 = 1.0 + log(u1 * (1.0 - e) + e) / alpha;
            ok = u2 * u2 <= 1.0 - y0 * y0;
        } else {
            // Kennedy-Pendleton: y0 = 1 - 2 lambda^2 with lambda^2 from a
            // three-dimensional Gaussian, accept with sqrt(1 - lambda^2)
            const double cs = cos(kTwoPi * u2);
            const double lam2 = -(log(u1) + cs * cs * log(u3)) / (2.0 * alpha);
            y0 = 1.0 - 2.0 * lam2;
            ok = u4 * u4 <= 1.0 - lam2;
        }
    }
    if (!ok) {
        y[0] = 1.0;
        y[1] = y[2] = y[3] = 0.0;
        return;
    }
    Ctr q = ctr;
    q.z |= 0xFFFFu;
    const Ctr r = philox4x32_10(q, k0, k1);
    const double ct = 2.0 * unit_open(r.x) - 1.0, ph = kTwoPi * unit_open(r.y);
    const double st = sqrt(fmax(0.0, 1.0 - ct * ct)), rad = sqrt(fmax(0.0, 1.0 - y0 * y0));
    y[0] = y0;
    y[1] = rad * st * cos(ph);
    y[2] = rad * st * sin(ph);
    y[3] = rad * ct;
}

// 2x2 SU(2) block of the unit quaternion x (layout of the file header)
struct Blk {
    cx<double> e[2][2];
};

__device__ __forceinline__ Blk quat_block(const double x[4]) {
    Blk m;
    m.e[0][0] = {x[0], x[3]};
    m.e[0][1] = {x[2], x[1]};
    m.e[1][0] = {-x[2], x[1]};
    m.e[1][1] = {x[0], -x[3]};
    return m;
}

__device__ __forceinline__ Blk blk_mul(const Blk &p, const Blk &q) {
    Blk r;
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++) r.e[i][j] = cmadd(cmul(p.e[i][0], q.e[0][j]), p.e[i][1], q.e[1][j]);
    return r;
}

// rows (RA, RB) of M <- A (rows RA, RB of M)
template <int RA, int RB>
__device__ __forceinline__ void rows_left_mul(M3<double> &M, const Blk &A) {
#pragma unroll
    for (int k = 0; k < 3; k++) {
        const cx<double> a = M.e[RA][k], b = M.e[RB][k];
        M.e[RA][k] = cmadd(cmul(A.e[0][0], a), A.e[0][1], b);
        M.e[RB][k] = cmadd(cmul(A.e[1][0], a), A.e[1][1], b);
    }
}

struct McArgs {
    const CfgDesc *cfgs;
    const int *tile_start;
    int n_cfg;
    int n_tiles;
    int par;          // 0: even sites, 1: odd sites
    int heatbath;     // 1: heat bath, 0: over-relaxation
    double beta;      // 18 b
    uint32_t k0, k1;  // Philox key (seed)
    uint32_t sweep;
};

template <int RA, int RB, int SUB>
__device__ __forceinline__ void subgroup_update(M3<double> &U, M3<double> &Om, const McArgs &a,
                                                int mu, int i, uint32_t cfg) {
    double c[4];
    c[0] = Om.e[RA][RA].x + Om.e[RB][RB].x;
    c[1] = -(Om.e[RA][RB].y + Om.e[RB][RA].y);
    c[2] = Om.e[RB][RA].x - Om.e[RA][RB].x;
    c[3] = Om.e[RB][RB].y - Om.e[RA][RA].y;
    const double k = sqrt(c[0] * c[0] + c[1] * c[1] + c[2] * c[2] + c[3] * c[3]);
    if (!(k > 1e-300)) return;
    const double inv = 1.0 / k;
    const double ch[4] = {c[0] * inv, c[1] * inv, c[2] * inv, c[3] * inv};
    const Blk C = quat_block(ch);
    Blk A;
    if (a.heatbath) {
        const Ctr ctr{(uint32_t)i, a.sweep, ((uint32_t)mu << 24) | ((uint32_t)SUB << 16), cfg};
        double y[4];
        su2_heatbath_draw(a.beta * k / 3.0, ctr, a.k0, a.k1, y);
        A = blk_mul(quat_block(y), C);
    } else {
        A = blk_mul(C, C);
    }
    rows_left_mul<RA, RB>(U, A);
    rows_left_mul<RA, RB>(Om, A);
}

template <int MU>
__device__ __forceinline__ void mc_link(const McArgs &a, const CfgDesc &c, int i) {
    void *base = c.cur ? c.W[1] : c.W[0];
    const Links<double, 9, true> W{as_global<double>((const void *)base), c.stride};
    const Geo g = make_geo(c, i);
    M3<double> S;
    m_zero(S);
#pragma unroll
    for (int nu = 0; nu < 4; nu++) {
        if (nu == MU) continue;
        m_acc(S, upper_staple(W, c, g, MU, nu));
        acc_lower_staple(S, W, c, g, MU, nu);
    }
    M3<double> U = W(MU, i);
    M3<double> Om = mul_nn(U, S);
    const uint32_t cfg = (uint32_t)c.user;
    subgroup_update<0, 1, 0>(U, Om, a, MU, i, cfg);
    subgroup_update<0, 2, 1>(U, Om, a, MU, i, cfg);
    subgroup_update<1, 2, 2>(U, Om, a, MU, i, cfg);
    store_link<double, 9, true>(as_global<double>(base), c.stride, MU, i, U);
}

// A wave takes 64 consecutive sites of one parity of one configuration:
// half-lattice index k -> row r = k / (d0/2) of sites along direction 0, and
// in that row the site 2 (k mod d0/2) + ((par + n1 + n2 + n3) mod 2).  The
// tile table counts V/2 sites per configuration; blocks are laid out
// XCD-contiguously.
template <int MU>
__global__ __launch_bounds__(256) void mc_kernel(McArgs a) {
    const int nb = (a.n_tiles + 3) >> 2;
    const int b = remap_block(blockIdx.x, nb, 1);
    if (b >= nb) return;
    const int tile = b * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (tile >= a.n_tiles) return;
    const int ci = find_cfg(a.tile_start, a.n_cfg, tile);
    const CfgDesc c = a.cfgs[ci];
    const int k = (tile - a.tile_start[ci]) * kTile + (threadIdx.x & 63);
    if (k >= (c.V >> 1)) return;
    const int h0 = c.d[0] >> 1;
    const int r = k / h0;
    const int j = k - r * h0;
    const int n1 = r % c.d[1];
    const int r2 = r / c.d[1];
    const int n2 = r2 % c.d[2];
    const int n3 = r2 / c.d[2];
    const int n0 = 2 * j + ((a.par + n1 + n2 + n3) & 1);
    mc_link<MU>(a, c, n0 + c.d[0] * r);
}

hipError_t launch_mc(hipStream_t s, const CfgDesc *cfgs, const int *tile_start, int n_cfg,
                     int n_tiles, int mu, int par, int heatbath, double beta, uint64_t seed,
                     uint32_t sweep) {
    if (n_tiles <= 0) return hipSuccess;
    McArgs a{cfgs, tile_start, n_cfg, n_tiles, par, heatbath, beta,
             (uint32_t)seed, (uint32_t)(seed >> 32), sweep};
    dim3 grid(((n_tiles + 3) / 4 + 7) / 8 * 8);
    switch (mu) {
        case 0: hipLaunchKernelGGL(mc_kernel<0>, grid, dim3(256), 0, s, a); break;
        case 1: hipLaunchKernelGGL(mc_kernel<1>, grid, dim3(256), 0, s, a); break;
        case 2: hipLaunchKernelGGL(mc_kernel<2>, grid, dim3(256), 0, s, a); break;
        default: hipLaunchKernelGGL(mc_kernel<3>, grid, dim3(256), 0, s, a); break;
    }
    return hipGetLastError();
}

}  // namespace tgf
