// sun_dev.h -- what the SU(N) kernels share (sun.hip: rows of a link in
// registers or LDS; sun_mfma.hip: products on the matrix cores): the link
// storage, twist phases, launch arguments, site groups and the plan of the
// exponential.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "launch.h"
#include "lattice_dev.h"
#include "layout.h"
#include "su3_dev.h"

namespace tgf {

// Storage of a link matrix, FP64 complex entries r N + j of link (mu, site):
// the N whose products run on the matrix cores keep a link together,
// [mu][site][entry], so that a wave reads whole links as contiguous 1 KB;
// the others, whose lanes hold rows or whole links of consecutive sites, keep
// the structure of arrays [mu][entry][site].
constexpr bool sun_aos(int n) { return n == 4 || n >= 7; }

template <int N>
__device__ __forceinline__ unsigned row_off(int r, int j, int stride, int site) {
    if constexpr (sun_aos(N)) return ((unsigned)site * (unsigned)(N * N) + (unsigned)(r * N + j)) * 16u;
    return ((unsigned)(r * N + j) * (unsigned)stride + (unsigned)site) * 16u;
}

// index of an entry in a link buffer
template <int N>
__device__ __forceinline__ size_t sun_index(int mu, int e, int stride, int i) {
    return sun_aos(N) ? ((size_t)mu * stride + i) * (N * N) + e : (size_t)(mu * N * N + e) * stride + i;
}

// twist exponent n_{mu nu} (mod N, antisymmetric) and Z = exp(2 pi i n / N)
template <int N>
__device__ __forceinline__ int tw_exp(const CfgDesc &c, int mu, int nu) {
    if (mu < nu) return c.tw[plane_index(mu, nu)];
    const int t = c.tw[plane_index(nu, mu)];
    return t ? N - t : 0;
}

// exp(2 pi i k / N) for N = 2..8, k = 0..N-1 as (cos, sin), the exact values
// rounded to double (evaluated to 60 digits; zeros and units exact).  A table
// read with a wave-uniform index keeps the trigonometric code, and the private
// memory its argument reduction uses, out of the flow kernels.
static __constant__ double kTwistPhase[9][8][2] = {
    {  // unused
        {0.0, 0.0}, {0.0, 0.0},
        {0.0, 0.0}, {0.0, 0.0},
        {0.0, 0.0}, {0.0, 0.0},
        {0.0, 0.0}, {0.0, 0.0},
    },
    {  // unused
        {0.0, 0.0}, {0.0, 0.0},
        {0.0, 0.0}, {0.0, 0.0},
        {0.0, 0.0}, {0.0, 0.0},
        {0.0, 0.0}, {0.0, 0.0},
    },
    {  // N = 2
        {1.0, 0.0}, {-1.0, 0.0},
        {0.0, 0.0}, {0.0, 0.0},
        {0.0, 0.0}, {0.0, 0.0},
        {0.0, 0.0}, {0.0, 0.0},
    },
    {  // N = 3
        {1.0, 0.0}, {-0.5, 0.8660254037844386},
        {-0.5, -0.8660254037844386}, {0.0, 0.0},
        {0.0, 0.0}, {0.0, 0.0},
        {0.0, 0.0}, {0.0, 0.0},
    },
    {  // N = 4
        {1.0, 0.0}, {0.0, 1.0},
        {-1.0, 0.0}, {0.0, -1.0},
        {0.0, 0.0}, {0.0, 0.0},
        {0.0, 0.0}, {0.0, 0.0},
    },
    {  // N = 5
        {1.0, 0.0}, {0.30901699437494745, 0.9510565162951535},
        {-0.8090169943749475, 0.5877852522924731}, {-0.8090169943749475, -0.5877852522924731},
        {0.30901699437494745, -0.9510565162951535}, {0.0, 0.0},
        {0.0, 0.0}, {0.0, 0.0},
    },
    {  // N = 6
        {1.0, 0.0}, {0.5, 0.8660254037844386},
        {-0.5, 0.8660254037844386}, {-1.0, 0.0},
        {-0.5, -0.8660254037844386}, {0.5, -0.8660254037844386},
        {0.0, 0.0}, {0.0, 0.0},
    },
    {  // N = 7
        {1.0, 0.0}, {0.6234898018587335, 0.7818314824680298},
        {-0.2225209339563144, 0.9749279121818236}, {-0.9009688679024191, 0.4338837391175581},
        {-0.9009688679024191, -0.4338837391175581}, {-0.2225209339563144, -0.9749279121818236},
        {0.6234898018587335, -0.7818314824680298}, {0.0, 0.0},
    },
    {  // N = 8
        {1.0, 0.0}, {0.7071067811865476, 0.7071067811865476},
        {0.0, 1.0}, {-0.7071067811865476, 0.7071067811865476},
        {-1.0, 0.0}, {-0.7071067811865476, -0.7071067811865476},
        {0.0, -1.0}, {0.7071067811865476, -0.7071067811865476},
    },
};

template <int N>
__device__ __forceinline__ cx<double> zphase(int t) {
    return {kTwistPhase[N][t][0], kTwistPhase[N][t][1]};
}

template <int N>
__device__ __forceinline__ cx<double> leaf_phase(const CfgDesc &c, int mu, int nu, int xm, int xn) {
    const int k = tw_exp<N>(c, mu, nu);
    if (k && xm == 0 && xn == 0) return cconj(zphase<N>(k));
    return {1.0, 0.0};
}

// The degree of the exponential's polynomial (expm1_blk in sun.hip).
struct ExpPlan {
    int q, s;
    double f;   // 2^-s
};
__device__ __forceinline__ ExpPlan exp_plan(double theta) {
    ExpPlan p{2, 0, 1.0};
    if (theta > 1.4) {
        p.s = min((int)ceil(log2(theta * (1.0 / 1.4))), 60);
        p.f = ldexp(1.0, -p.s);
        theta *= p.f;
    }
    p.q = theta <= 0.059 ? 2 : theta <= 0.21 ? 3 : theta <= 0.49 ? 4 : theta <= 0.88 ? 5 : 6;
    return p;
}
static __constant__ double kInvFact[21] = {
    1.0, 1.0, 1.0 / 2, 1.0 / 6, 1.0 / 24, 1.0 / 120, 1.0 / 720, 1.0 / 5040, 1.0 / 40320,
    1.0 / 362880, 1.0 / 3628800, 1.0 / 39916800, 1.0 / 479001600, 1.0 / 6227020800,
    1.0 / 87178291200, 1.0 / 1307674368000, 1.0 / 20922789888000, 1.0 / 355687428096000,
    1.0 / 6402373705728000, 1.0 / 121645100408832000, 1.0 / 2432902008176640000};

struct SunStageArgs {
    const CfgDesc *cfgs;
    const int *tile_start;
    int n_act;
    int n_tiles;
    int step;
    int stage;
    double eps;
};

static __constant__ double kSunRkA[3] = {0.0, -17.0 / 9.0, -1.0};
static __constant__ double kSunRkB[3] = {0.25, 8.0 / 9.0, 0.75};

// sun_mfma.hip: the matrix-core variants (nc = 4, 7, 8)
hipError_t launch_stage_sun_mfma(int nc, hipStream_t s, const SunStageArgs &a);
hipError_t launch_measure_sun_mfma(int nc, hipStream_t s, const CfgDesc *cfgs,
                                   const int *tile_start, int n_cfg, int n_tiles,
                                   const MeasSlot *slots, double *partials, int buf_sel);

// Site groups of the stage launches.  A wave holds G = 64 / L sites; the sites
// of a configuration are cut into groups of G, and every group is a work-group
// of its own (wave w updates direction w).  ceil(64 / G) work-groups are
// launched per 64-site tile, enough for every group of the configuration; the
// few past its end return.  One group per work-group, not a loop over a tile's
// groups: a 3x3x15x15 SU(5) box is 169 work-groups of one group instead of 32
// of six in a row (a 16-step flow 7.2 -> 1.8 ms; 4x4x20x20 boxes of 102k sites
// -19%), and no group is cut at a tile's end.  The launch order gives each XCD
// one contiguous range of groups.
template <int G>
struct SiteGroups {
    static constexpr int P = (kTile + G - 1) / G;   // work-groups per tile
};

// site of lane 0 of the group that work-group b takes (-1: none) and its configuration
template <int G>
__device__ __forceinline__ int group_first(const SunStageArgs &a, int &ci) {
    constexpr int P = SiteGroups<G>::P;
    const int nb = a.n_tiles * P;
    const int b = remap_block(blockIdx.x, nb, 1);
    if (b >= nb) return -1;
    const int tile = b / P;
    ci = find_cfg(a.tile_start, a.n_act, tile);
    const int first = (b - a.tile_start[ci] * P) * G;
    return first < a.cfgs[ci].V ? first : -1;
}

__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

}  // namespace tgf
