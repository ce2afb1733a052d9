// sun_mfma.hip -- the SU(N) flow stage and measurement with the N x N products
// on the matrix cores (v_mfma_f64_4x4x4_4b_f64), FP64, N = 4, 7 and 8, gfx950.
// The method is that of sun.hip.
//
// One instruction multiplies four independent pairs of 4 x 4 matrices, one
// double per lane and operand.  With lane = c + 4 b + 16 r (b the block):
//   B and D operands   hold entry (r, c) of block b ("natural" layout),
//   the A operand      holds entry (c, r) of block b.
// N = 4: the four blocks are four sites.  N = 7, 8: the four blocks (I, J),
// b = 2 I + J, are the quarters of one 8 x 8 matrix (N = 7 padded with zeros),
// and a product takes two steps: D_IJ += A_II B_IJ, then D_IJ += A_I(1-I)
// B_(1-I)J, whose right operand is the natural register with lanes l and
// l ^ 8 exchanged.  A complex product is four real ones (signs by the
// instruction's negate bit).
//
// Every product of a stage is written so that its left operand is a link (read
// from memory straight into the A layout, or that of its adjoint) or a power
// of an anti-Hermitian matrix: a natural register read as A gives the
// transpose, which for X^+ = +-X is +-conj(X), so those need no exchange of
// lanes (N = 4) or one within 16 lanes (N = 8).  Sums of staples and the
// polynomial's additions ride in the C operand.
//
// Why: FP64 matrix instructions and FP64 vector FMAs have the same peak here
// (62-65 and 60 TFLOP/s measured, and they share the unit), so what the matrix
// cores save is operand traffic.  With rows of a link in lanes, every complex
// multiply-add needs an operand fetched from LDS (N = 8: the LDS pipe was the
// limit at 24 TFLOP/s) or whole matrices in registers (N = 4: 408 registers,
// one wave per SIMD).  Here a complex matrix is four registers per lane and an
// operand is read once per product.  A wave works on the four links of its
// sites, so an upper plaquette serves both of its links: 46 products of
// staples and 20 of the exponential and update per site and stage, against 52
// and 48 (20 with this polynomial).
//
// Stage launch, MI355X, against the rows-in-lanes kernels before: SU(4)
// 4x4x16x16 x 48 (197k sites) 386 -> 228 us; SU(7) 4x4x28x28 x 6 (75k) 1097 ->
// 596 us; SU(8) 4x4x32x32 x 4 (66k) 1198 -> 481 us.  The matrix instructions'
// own time is 0.225 ms of the last (66 products x 8 instructions x 16 cycles per
// site on 1024 SIMDs at 2.4 GHz): the rest is waiting for operands, an adjoint
// being read as two overlapping blocks.  SU(4) is held by issue: 264 matrix and
// about 600 other vector instructions per wave of four sites (680 MB per launch,
// no refetch; 85 us of matrix time).  Measurement of the same boxes: 433 -> 291,
// 1098 -> 630, 1463 -> 672 us.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "launch.h"
#include "lattice_dev.h"
#include "layout.h"
#include "su3_dev.h"
#include "sun_dev.h"

namespace tgf {

// one complex matrix (N = 4: four of them), one entry per lane
struct Zm {
    double r, i;
};

template <int N>
struct Mx {
    static constexpr int B = N > 4 ? 2 : 1;    // 4 x 4 blocks per matrix and dimension
    static constexpr int G = N > 4 ? 1 : 4;    // sites per wave
    static constexpr bool kPad = N != 4 * B;   // lanes outside the matrix hold zeros
};

// A operand: step 0 the block (I, I), step 1 the block (I, 1 - I)
template <int N>
struct AOp {
    Zm s[Mx<N>::B];
};

// this lane's entries, as element offsets in a link matrix (row-major, N^2)
template <int N>
struct LaneMap {
    int nat, tr;               // natural entry, and its transpose
    int a[Mx<N>::B];           // A layout of X: entry read for step k
    int ad[Mx<N>::B];          // A layout of X^+: entry of X, conjugated
    bool in_nat, in_a[Mx<N>::B];   // inside the matrix (N = 7)
    bool diag;
    int t_lane;                // lane that holds the transposed entry
};

template <int N>
__device__ __forceinline__ LaneMap<N> lane_map() {
    const int l = threadIdx.x & 63;
    const int c = l & 3, b = (l >> 2) & 3, r = l >> 4;
    LaneMap<N> m;
    if constexpr (Mx<N>::B == 1) {
        m.nat = r * 4 + c;
        m.tr = c * 4 + r;
        m.a[0] = m.tr;
        m.ad[0] = m.nat;
        m.in_nat = m.in_a[0] = true;
        m.diag = r == c;
        m.t_lane = r + 4 * b + 16 * c;
    } else {
        const int I = b >> 1, J = b & 1;
        const int R = 4 * I + r, C = 4 * J + c;
        m.in_nat = R < N && C < N;
        m.nat = R * N + C;
        m.tr = C * N + R;
#pragma unroll
        for (int k = 0; k < 2; k++) {
            const int row = 4 * I + c, col = 4 * (k ? 1 - I : I) + r;
            m.in_a[k] = row < N && col < N;
            m.a[k] = row * N + col;
            m.ad[k] = col * N + row;
        }
        m.diag = R == C && m.in_nat;
        m.t_lane = r + 4 * (2 * J + I) + 16 * c;
    }
    return m;
}

template <int N>
__device__ __forceinline__ Zm ld_entry(gptr<const v2<double>> W, int site, int e, bool in) {
    const unsigned off = ((unsigned)site * (unsigned)(N * N) + (unsigned)(Mx<N>::kPad && !in ? 0 : e)) * 16u;
    const cx<double> v = ld(W, off);
    if constexpr (Mx<N>::kPad) return in ? Zm{v.x, v.y} : Zm{0.0, 0.0};
    return {v.x, v.y};
}

// links of direction mu start here
template <int N>
__device__ __forceinline__ gptr<const v2<double>> dir_base(gptr<const v2<double>> W, int stride,
                                                           int mu) {
    return W + (size_t)(mu * N * N) * stride;
}

// natural layout of U and of U^+
template <int N>
__device__ __forceinline__ Zm ld_nat(gptr<const v2<double>> W, const LaneMap<N> &m, int site) {
    return ld_entry<N>(W, site, m.nat, m.in_nat);
}
template <int N>
__device__ __forceinline__ Zm ld_nat_dag(gptr<const v2<double>> W, const LaneMap<N> &m, int site) {
    const Zm z = ld_entry<N>(W, site, m.tr, m.in_nat);
    return {z.r, -z.i};
}
// A layout of U; of conj(U^+) (multiply with kConj)
template <int N>
__device__ __forceinline__ AOp<N> ld_a(gptr<const v2<double>> W, const LaneMap<N> &m, int site) {
    AOp<N> o;
#pragma unroll
    for (int k = 0; k < Mx<N>::B; k++) o.s[k] = ld_entry<N>(W, site, m.a[k], m.in_a[k]);
    return o;
}
template <int N>
__device__ __forceinline__ AOp<N> ld_ad(gptr<const v2<double>> W, const LaneMap<N> &m, int site) {
    AOp<N> o;
#pragma unroll
    for (int k = 0; k < Mx<N>::B; k++) o.s[k] = ld_entry<N>(W, site, m.ad[k], m.in_a[k]);
    return o;
}

template <int kCtrl, int kBank>
__device__ __forceinline__ double dpp_d(double old, double src) {
    const uint64_t o = __builtin_bit_cast(uint64_t, old), s = __builtin_bit_cast(uint64_t, src);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)o, (int)(uint32_t)s, kCtrl, 0xf, kBank, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)(o >> 32), (int)(uint32_t)(s >> 32), kCtrl, 0xf, kBank, false);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
// DPP controls within a row of 16 lanes (four banks of 4 lanes = the blocks b)
constexpr int kRowShl4 = 0x104, kRowShl8 = 0x108, kRowShr4 = 0x114, kRowShr8 = 0x118, kRowRor8 = 0x128;

// The natural register v read as an A operand (its transpose): step k needs
// X_II and X_(1-I)I in the blocks (I, J).
template <int N>
__device__ __forceinline__ AOp<N> a_of_nat(const Zm &v) {
    AOp<N> o;
    if constexpr (Mx<N>::B == 1) {
        o.s[0] = v;
    } else {
        auto step0 = [](double x) {
            double y = dpp_d<kRowShr4, 0x2>(x, x);      // block (0,1) from (0,0)
            return dpp_d<kRowShl4, 0x4>(y, x);          // block (1,0) from (1,1)
        };
        auto step1 = [](double x) {
            double y = dpp_d<kRowShl8, 0x1>(x, x);      // (0,0) from (1,0)
            y = dpp_d<kRowShl4, 0x2>(y, x);             // (0,1) from (1,0)
            y = dpp_d<kRowShr4, 0x4>(y, x);             // (1,0) from (0,1)
            return dpp_d<kRowShr8, 0x8>(y, x);          // (1,1) from (0,1)
        };
        o.s[0] = {step0(v.r), step0(v.i)};
        o.s[1] = {step1(v.r), step1(v.i)};
    }
    return o;
}

template <int kNeg>
__device__ __forceinline__ double mfma4(double a, double b, double c) {
    return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, kNeg);
}

// c + s A b; kConj: A stands for conj of the register, kNeg: s = -1
template <int N, bool kConj, bool kNeg = false>
__device__ __forceinline__ Zm mul(const AOp<N> &A, const Zm &b, Zm c) {
    constexpr int P = kNeg ? 1 : 0, Q = kNeg ? 0 : 1;   // sign of A_r products; its opposite
#pragma unroll
    for (int k = 0; k < Mx<N>::B; k++) {
        Zm x = b;
        if (k) x = {dpp_d<kRowRor8, 0xf>(b.r, b.r), dpp_d<kRowRor8, 0xf>(b.i, b.i)};
        c.r = mfma4<P>(A.s[k].r, x.r, c.r);
        c.i = mfma4<P>(A.s[k].r, x.i, c.i);
        c.r = mfma4<kConj ? P : Q>(A.s[k].i, x.i, c.r);
        c.i = mfma4<kConj ? Q : P>(A.s[k].i, x.r, c.i);
    }
    return c;
}

__device__ __forceinline__ Zm zm_add(const Zm &a, const Zm &b) { return {a.r + b.r, a.i + b.i}; }

// M^+ of a natural register
template <int N>
__device__ __forceinline__ Zm dagger(const Zm &v, const LaneMap<N> &m) {
    return {__shfl(v.r, m.t_lane), -__shfl(v.i, m.t_lane)};
}

// sum over the entries of a matrix (16 or 64 lanes)
template <int N>
__device__ __forceinline__ double mat_sum(double v) {
    v += __shfl_xor(v, 1);
    v += __shfl_xor(v, 2);
    v += __shfl_xor(v, 16);
    v += __shfl_xor(v, 32);
    if constexpr (Mx<N>::B == 2) {
        v += __shfl_xor(v, 4);
        v += __shfl_xor(v, 8);
    }
    return v;
}
// largest over the matrices of the wave (v uniform over a matrix)
template <int N>
__device__ __forceinline__ double wave_most(double v) {
    if constexpr (Mx<N>::B == 1) {
        v = fmax(v, __shfl_xor(v, 4));
        v = fmax(v, __shfl_xor(v, 8));
    }
    return v;
}

// exp(-X) - 1 for four anti-Hermitian natural registers X (the polynomial and
// degrees of expm1_blk in sun.hip), side by side so that four chains of matrix
// instructions are in flight.  All take the degree of the largest norm in the
// wave: the matrix instructions work on every block of it, whatever lanes are
// active.
template <int N>
__device__ __forceinline__ void expm1_neg(Zm (&x)[4], const LaneMap<N> &m, Zm (&t)[4]) {
    double n2 = 0.0;
#pragma unroll
    for (int q = 0; q < 4; q++) n2 = fmax(n2, mat_sum<N>(fma(x[q].r, x[q].r, x[q].i * x[q].i)));
    ExpPlan pl = exp_plan(sqrt(wave_most<N>(n2)));
    pl.q = __builtin_amdgcn_readfirstlane(pl.q);
    pl.s = __builtin_amdgcn_readfirstlane(pl.s);
    const Zm zero = {0.0, 0.0};
    Zm x2[4];
    AOp<N> a3[4];
#pragma unroll
    for (int q = 0; q < 4; q++) {
        if (pl.s) x[q] = {pl.f * x[q].r, pl.f * x[q].i};
        // a natural X read as A is -conj(X): X M = -conj(A) M
        const AOp<N> ax = a_of_nat<N>(x[q]);
        x2[q] = mul<N, true, true>(ax, x[q], zero);
        a3[q] = a_of_nat<N>(mul<N, true, true>(ax, x2[q], zero));
    }
    auto poly = [&](int q, double k0, double k1, double k2) {   // k0 - k1 X + k2 X^2
        Zm o = {fma(k2, x2[q].r, -k1 * x[q].r), fma(k2, x2[q].i, -k1 * x[q].i)};
        if (m.diag) o.r += k0;
        return o;
    };
    const double *k = kInvFact + 3 * pl.q;
#pragma unroll
    for (int q = 0; q < 4; q++) t[q] = poly(q, k[0], k[1], k[2]);
    for (int j = pl.q - 1; j >= 0; j--) {
        k = kInvFact + 3 * j;
        const double k0 = j ? k[0] : 0.0, k1 = k[1], k2 = k[2];
#pragma unroll
        for (int q = 0; q < 4; q++) t[q] = mul<N, true>(a3[q], t[q], poly(q, k0, k1, k2));   // - X^3 t
    }
    for (int i = 0; i < pl.s; i++)
#pragma unroll
        for (int q = 0; q < 4; q++) {
            // (1 + t)^2 - 1; the adjoint's natural register read as A is conj(t)
            const Zm d = {2.0 * t[q].r, 2.0 * t[q].i};
            t[q] = mul<N, true>(a_of_nat<N>(dagger<N>(t[q], m)), t[q], d);
        }
}

// z a on the lanes where `on`, else a
__device__ __forceinline__ Zm zm_scale_if(const Zm &a, cx<double> z, bool on) {
    const double x = on ? z.x : 1.0, y = on ? z.y : 0.0;
    return {fma(a.r, x, -a.i * y), fma(a.r, y, a.i * x)};
}

// sites of this wave's group, clamped into the configuration: `live` is false
// on lanes of a site past the end (their blocks compute, and store nothing)
template <int N>
__device__ __forceinline__ int wave_site(int first, int V, bool &live) {
    const int b = Mx<N>::B == 1 ? (int)((threadIdx.x >> 2) & 3) : 0;
    const int i = first + b;
    live = i < V;
    return live ? i : V - 1;
}

// Twist phases Z_{mu nu} of the six planes.  kAll = false: only plane (0, 1)
// is twisted (the scheme's own setting), the others' factors are known to be 1
// and cost nothing.  No branch stands between the loads of one staple and the
// next, so that they are issued well ahead of the products: with a branch per
// factor the compiler left one load in flight (SU(4) stage launch 277 us, now
// 235; SU(8) 595, now 499).
template <int N, bool kAll>
struct Phases {
    cx<double> z[6];
    __device__ __forceinline__ explicit Phases(const CfgDesc &c) {
#pragma unroll
        for (int p = 0; p < (kAll ? 6 : 1); p++) z[p] = zphase<N>(c.tw[p]);
    }
    // Z_{mu nu} a where `on`, or its conjugate
    __device__ __forceinline__ Zm scale(const Zm &a, int mu, int nu, bool on, bool conj) const {
        const int p = mu < nu ? plane_index(mu, nu) : plane_index(nu, mu);
        if (!kAll && p) return a;
        cx<double> w = z[p];
        if (conj != (mu > nu)) w.y = -w.y;
        return zm_scale_if(a, w, on);
    }
};

// the flow stage of one wave's sites, all four links
template <int N, bool kAll>
__device__ __forceinline__ void stage_body(const SunStageArgs &a, const CfgDesc &c, int first) {
    bool live;
    const int i = wave_site<N>(first, c.V, live);
    const Geo g = make_geo(c, i);
    const LaneMap<N> m = lane_map<N>();
    const Phases<N, kAll> ph(c);
    const int in = (c.cur + 3 * a.step + a.stage) & 1;
    gptr<const v2<double>> W = as_global<double>((const void *)(in ? c.W[1] : c.W[0]));
    gptr<v2<double>> Wout = as_global<double>(in ? c.W[0] : c.W[1]);
    gptr<v2<double>> X = as_global<double>(c.X);
    const int st = c.stride;
    const Zm zero = {0.0, 0.0};
    gptr<const v2<double>> D[4];
    AOp<N> U[4];
    Zm S[4], Om[4];
#pragma unroll
    for (int mu = 0; mu < 4; mu++) {
        D[mu] = dir_base<N>(W, st, mu);
        S[mu] = Om[mu] = zero;
    }
    // Eighteen staples, two products each with the left operands P, Q and the
    // right operand R:
    //   0..5   upper staple of link mu < nu, V = U_nu(n+mu) U_mu(n+nu)^+ U_nu(n)^+ Z^*;
    //          the plaquette U_mu V is minus what link nu gets (P_ah(P^+) = -P_ah(P));
    //   6..17  lower staple U_nu(n+mu-nu)^+ U_mu(n-nu)^+ U_nu(n-nu) Z.
    // The operands of staple s + kAhead are requested before staple s is
    // multiplied, and the fence keeps the compiler from sinking the requests
    // back to their use (left alone it kept one load in flight).  Two ahead at
    // three waves per SIMD; one or three ahead, or four waves: SU(8) 601, 503
    // and 634 us, SU(4) within 3%.
    constexpr int kAhead = 2;
    constexpr int kMu[18] = {0, 0, 1, 0, 1, 2, 1, 2, 3, 0, 2, 3, 0, 1, 3, 0, 1, 2};
    constexpr int kNu[18] = {1, 2, 2, 3, 3, 3, 0, 0, 0, 1, 1, 1, 2, 2, 2, 3, 3, 3};
    AOp<N> P[18], Q[18];
    Zm R[18], z[4], u[4];
    auto request = [&](int s) {
        const int mu = kMu[s], nu = kNu[s];
        const bool upper = s < 6;
        const int j = upper ? i : i + g.dn(nu);
        if (s && kNu[s - 1] == nu) R[s] = R[s - 1];
        else R[s] = upper ? ld_nat_dag<N>(D[nu], m, i) : ld_nat<N>(D[nu], m, j);
        P[s] = ld_ad<N>(D[mu], m, upper ? i + g.up(nu) : j);
        Q[s] = upper ? ld_a<N>(D[nu], m, i + g.up(mu)) : ld_ad<N>(D[nu], m, j + g.up(mu));
    };
#pragma unroll
    for (int mu = 0; mu < 3; mu++) U[mu] = ld_a<N>(D[mu], m, i);
#pragma unroll
    for (int s = 0; s < kAhead; s++) request(s);
#pragma unroll
    for (int s = 0; s < 18; s++) {
        const int mu = kMu[s], nu = kNu[s];
        if (s + kAhead < 18) request(s + kAhead);
        if (s == 6) U[3] = ld_a<N>(D[3], m, i);
        if (s == 16) {
#pragma unroll
            for (int q = 0; q < 4; q++) {
                z[q] = a.stage > 0 ? ld_nat<N>((gptr<const v2<double>>)X + (size_t)(q * N * N) * st, m, i) : zero;
                u[q] = ld_nat<N>(D[q], m, i);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if (s < 6) {
            Zm v = ph.scale(R[s], mu, nu, g.n(mu) == 0 && g.n(nu) == 0, true);
            v = mul<N, true>(P[s], v, zero);
            v = mul<N, false>(Q[s], v, zero);
            S[mu] = zm_add(S[mu], v);
            Om[nu] = mul<N, false, true>(U[mu], v, Om[nu]);
        } else {
            Zm v = ph.scale(R[s], mu, nu, g.n(mu) == 0 && g.back(nu) == 0, false);
            v = mul<N, true>(P[s], v, zero);
            S[mu] = mul<N, true>(Q[s], v, S[mu]);
        }
    }
    const double eps = a.step < c.n_full ? a.eps : c.eps_last;
    const double beps = -kSunRkB[a.stage] * eps, ac = kSunRkA[a.stage];
    const unsigned off = ((unsigned)i * (unsigned)(N * N) + (unsigned)m.nat) * 16u;
    const bool mine = live && m.in_nat;
    Zm e[4];
#pragma unroll
    for (int mu = 0; mu < 4; mu++) {
        const Zm om = mul<N, false>(U[mu], S[mu], Om[mu]);
        const Zm od = dagger<N>(om, m);
        const double t = mat_sum<N>(m.diag ? om.i : 0.0) / (double)N;
        // B eps F + A X, F = -P_ah(Omega)
        z[mu] = {fma(ac, z[mu].r, 0.5 * beps * (om.r - od.r)),
                 fma(ac, z[mu].i, beps * (0.5 * (om.i - od.i) - (m.diag ? t : 0.0)))};
    }
    if (a.stage < 2 && mine)
#pragma unroll
        for (int mu = 0; mu < 4; mu++)
            st_nt(X + (size_t)(mu * N * N) * st, off, cx<double>{z[mu].r, z[mu].i});
    // exp(X) U = U + (exp(X) - 1) U: the natural register of exp(-X) - 1 read
    // as A is conj(exp(X) - 1)
    expm1_neg<N>(z, m, e);
#pragma unroll
    for (int mu = 0; mu < 4; mu++) {
        const Zm n = zm_add(u[mu], mul<N, true>(a_of_nat<N>(e[mu]), u[mu], zero));
        if (mine) st_nt(Wout + (size_t)(mu * N * N) * st, off, cx<double>{n.r, n.i});
    }
}

__device__ __forceinline__ bool only_plane01(const CfgDesc &c) {
    return (c.tw[1] | c.tw[2] | c.tw[3] | c.tw[4] | c.tw[5]) == 0;
}

// One wave per group of G sites; a work-group holds four consecutive groups.
template <int N>
__global__ __launch_bounds__(256, 3) void sun_stage_mfma_kernel(SunStageArgs a) {
    constexpr int G = Mx<N>::G;
    int ci = 0;
    const int wg_first = group_first<4 * G>(a, ci);
    if (wg_first < 0) return;
    const CfgDesc &c = a.cfgs[ci];   // in global memory, like the other SU(N) kernels
    const int first = wg_first + G * __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (first >= c.V) return;
    if (only_plane01(c))
        stage_body<N, false>(a, c, first);
    else
        stage_body<N, true>(a, c, first);
}

// The measurement.  G depends on the leaf sum only through C - C^+, so leaves
// 2 and 3 enter through their adjoints, which share a factor with leaves 1
// and 4:
//   M = U_mu(n) [V - L] + U_mu(n-mu)^+ [Y - Q],   C - C^+ = M - M^+,
//   V = U_nu(n+mu) U_mu(n+nu)^+ U_nu(n)^+            (leaf 1 = U_mu V)
//   L = U_nu(n+mu-nu)^+ U_mu(n-nu)^+ U_nu(n-nu)      (leaf 2^+ = U_mu L)
//   Q = U_nu(n-mu) U_mu(n-mu+nu) U_nu(n)^+           (leaf 3^+ = U_mu(n-mu)^+ Q)
//   Y = U_nu(n-mu-nu)^+ U_mu(n-mu-nu) U_nu(n-nu)     (leaf 4 = U_mu(n-mu)^+ Y)
// each with its twist factor: ten products per plane, not twelve.  Returns
// this lane's entry of G; rp += its share of Re Tr of leaf 1.
template <int N>
__device__ __forceinline__ Zm clover_mx(gptr<const v2<double>> W, const CfgDesc &c, const Geo &g,
                                        const LaneMap<N> &m, const Phases<N, true> &ph, int mu,
                                        int nu, double &rp) {
    gptr<const v2<double>> Dm = dir_base<N>(W, c.stride, mu), Dn = dir_base<N>(W, c.stride, nu);
    const int i = g.i, j = i + g.dn(nu), h = i + g.dn(mu), hj = h + g.dn(nu);
    const bool m0 = g.n(mu) == 0, n0 = g.n(nu) == 0, mb = g.back(mu) == 0, nb = g.back(nu) == 0;
    const Zm zero = {0.0, 0.0};
    const Zm ud = ld_nat_dag<N>(Dn, m, i);
    const Zm un = ld_nat<N>(Dn, m, j);
    Zm v = ph.scale(ud, mu, nu, m0 && n0, true);
    v = mul<N, true>(ld_ad<N>(Dm, m, i + g.up(nu)), v, zero);
    v = mul<N, false>(ld_a<N>(Dn, m, i + g.up(mu)), v, zero);
    const Zm um = ld_nat_dag<N>(Dm, m, i);   // conj of the transposed entry
    rp = fma(um.r, v.r, fma(um.i, v.i, rp));
    Zm t = ph.scale(un, mu, nu, m0 && nb, false);
    t = mul<N, true>(ld_ad<N>(Dm, m, j), t, zero);
    v = mul<N, true, true>(ld_ad<N>(Dn, m, j + g.up(mu)), t, v);
    Zm M = mul<N, false>(ld_a<N>(Dm, m, i), v, zero);
    t = ph.scale(un, mu, nu, mb && nb, true);
    t = mul<N, false>(ld_a<N>(Dm, m, hj), t, zero);
    v = mul<N, true>(ld_ad<N>(Dn, m, hj), t, zero);
    t = ph.scale(ud, mu, nu, mb && n0, false);
    t = mul<N, false>(ld_a<N>(Dm, m, h + g.up(nu)), t, zero);
    v = mul<N, false, true>(ld_a<N>(Dn, m, h), t, v);
    M = mul<N, true>(ld_ad<N>(Dm, m, h), v, M);
    // G = -(i/8)(M - M^+)
    const Zm md = dagger<N>(M, m);
    return {0.125 * (M.i - md.i), -0.125 * (M.r - md.r)};
}

// A tile's 64 / G groups are dealt to three work-groups (partial slots) of W
// waves, K groups one after another in a wave.  Each XCD takes a run of
// every configuration's tiles (48 boxes 4x4x16x16 of SU(4) 311 -> 293 us).
template <int N>
struct MxMeas {
    static constexpr int P = kTile / Mx<N>::G;
    static constexpr int W = N == 4 ? 6 : 8;
    static constexpr int K = (P + 3 * W - 1) / (3 * W);
};

template <int N>
__global__ __launch_bounds__(64 * MxMeas<N>::W) void sun_measure_mfma_kernel(
    const CfgDesc *__restrict__ cfgs, const int *__restrict__ tile_start, int n_cfg, int n_tiles,
    const MeasSlot *__restrict__ slots, double *__restrict__ partials, int buf_sel) {
    constexpr int G = Mx<N>::G, W = MxMeas<N>::W, K = MxMeas<N>::K;
    const int ci = find_cfg(tile_start, n_cfg, blockIdx.x / 3);
    if (slots[ci].row < 0) return;
    const CfgDesc &c = cfgs[ci];
    const int b = run_order(blockIdx.x - 3 * tile_start[ci], 3 * ((c.V + kTile - 1) / kTile));
    const int tile = tile_start[ci] + b / 3, slot = b % 3;
    const int sel = buf_sel < 0 ? c.cur : ((c.cur + buf_sel) & 1);
    gptr<const v2<double>> L = as_global<double>((const void *)(sel ? c.W[1] : c.W[0]));
    const int t0 = (tile - tile_start[ci]) * kTile;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const LaneMap<N> m = lane_map<N>();
    const Phases<N, true> ph(c);
    double v[4] = {0, 0, 0, 0};
#pragma unroll 1
    for (int k = 0; k < K; k++) {
        const int s0 = ((k * 3 + slot) * W + w) * G;
        const int first = t0 + s0;
        if (s0 >= kTile || first >= c.V) break;          // whole wave
        bool live;
        const Geo g = make_geo(c, wave_site<N>(first, c.V, live));
        double e = 0.0, q = 0.0, p = 0.0;
#pragma unroll
        for (int pr = 0; pr < 3; pr++) {
            const int a1 = pr + 1;                         // planes (0, a1) and (b0, b1)
            const int b0 = pr == 0 ? 2 : 1, b1 = pr == 2 ? 2 : 3;
            const Zm Ga = clover_mx<N>(L, c, g, m, ph, 0, a1, p);
            const Zm Gb = clover_mx<N>(L, c, g, m, ph, b0, b1, p);
            e = fma(Ga.r, Ga.r, fma(Ga.i, Ga.i, fma(Gb.r, Gb.r, fma(Gb.i, Gb.i, e))));
            const double d = fma(Ga.r, Gb.r, Ga.i * Gb.i);
            q += pr == 1 ? -d : d;
        }
        if (live) {
            v[0] += e;
            v[1] += q * 0.025330295910584444;   // 1 / (4 pi^2)
            v[2] += p;
            v[3] += (m.diag ? 6.0 : 0.0) - p;
        }
    }
    __shared__ double red[W][4];
#pragma unroll
    for (int k = 0; k < 4; k++) v[k] = wave_sum_d(v[k]);
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int k = 0; k < 4; k++) red[w][k] = v[k];
    __syncthreads();
    if (threadIdx.x < 4) {
        double t = red[0][threadIdx.x];
#pragma unroll
        for (int x = 1; x < W; x++) t += red[x][threadIdx.x];
        partials[((size_t)tile * 3 + slot) * 4 + threadIdx.x] = t;
    }
}

// ---------------------------------------------------------------------------
// launchers

template <int N>
static hipError_t stage_n(hipStream_t s, const SunStageArgs &a) {
    const dim3 grid((a.n_tiles * SiteGroups<4 * Mx<N>::G>::P + 7) / 8 * 8);
    hipLaunchKernelGGL((sun_stage_mfma_kernel<N>), grid, dim3(256), 0, s, a);
    return hipGetLastError();
}
hipError_t launch_stage_sun_mfma(int nc, hipStream_t s, const SunStageArgs &a) {
    return nc == 4 ? stage_n<4>(s, a) : nc == 7 ? stage_n<7>(s, a)
         : nc == 8 ? stage_n<8>(s, a) : hipErrorInvalidValue;
}

template <int N>
static hipError_t measure_n(hipStream_t s, const CfgDesc *cfgs, const int *tile_start, int n_cfg,
                            int n_tiles, const MeasSlot *slots, double *partials, int buf_sel) {
    hipLaunchKernelGGL((sun_measure_mfma_kernel<N>), dim3(3 * n_tiles), dim3(64 * MxMeas<N>::W), 0,
                       s, cfgs, tile_start, n_cfg, n_tiles, slots, partials, buf_sel);
    return hipGetLastError();
}
hipError_t launch_measure_sun_mfma(int nc, hipStream_t s, const CfgDesc *cfgs,
                                   const int *tile_start, int n_cfg, int n_tiles,
                                   const MeasSlot *slots, double *partials, int buf_sel) {
    return nc == 4   ? measure_n<4>(s, cfgs, tile_start, n_cfg, n_tiles, slots, partials, buf_sel)
           : nc == 7 ? measure_n<7>(s, cfgs, tile_start, n_cfg, n_tiles, slots, partials, buf_sel)
           : nc == 8 ? measure_n<8>(s, cfgs, tile_start, n_cfg, n_tiles, slots, partials, buf_sel)
                     : hipErrorInvalidValue;
}

}  // namespace tgf
