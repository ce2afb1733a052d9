// Host audit of the quad stage kernel's index arithmetic (test
// infrastructure), with the kernel's own index functions.
//
//  - make_geo_inv, whose divisions are products with 1/d, gives make_geo's
//    coordinates: on every site of small boxes, and on the sites around every
//    multiple of each divisor's block near the ends and at random of boxes up
//    to the site cap (2^28 - 256).
//  - The column order of a large box's tiles is a one-to-one map.
//  - Every tile of 64 sites: where all lanes find n - 0, n - 1, n + 0 or n + 1
//    in the tile, those are slots of the tile that hold that site; the sites
//    of the lanes past the end are the last one; and a wave's lanes that take a
//    conjugated form from a closed tile read each slot exactly once.
#include <hip/hip_runtime.h>

#include <array>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "lattice_dev.h"
#include "layout.h"

using namespace tgf;

static long long checked = 0, bad = 0;
static void fail(const char *what, const CfgDesc &c, long long i) {
    if (bad < 20)
        std::fprintf(stderr, "violation: %s %dx%dx%dx%d site %lld\n", what, c.d[0], c.d[1], c.d[2],
                     c.d[3], i);
    bad++;
}

static CfgDesc desc(const std::array<int, 4> &d) {
    CfgDesc c{};
    c.V = 1;
    for (int m = 0; m < 4; m++) {
        c.d[m] = d[m];
        c.V *= d[m];
    }
    for (int m = 0; m < 3; m++) c.inv[m] = 1.0 / d[m];
    c.stride = (c.V + 255) / 256 * 256;
    return c;
}

static void same(const CfgDesc &c, int i) {
    if (i < 0 || i >= c.V) return;
    checked++;
    const Geo a = make_geo(c, i), b = make_geo_inv(c, i);
    if (a.n0 != b.n0 || a.n1 != b.n1 || a.n2 != b.n2 || a.n3 != b.n3 || a.i != b.i || a.s1 != b.s1 ||
        a.s2 != b.s2 || a.s3 != b.s3)
        fail("coordinates", c, i);
}

static void tiles(const CfgDesc &c) {
    for (int tb = 0; tb < c.V; tb += kTile) {
        const int nw = c.V - tb < kTile ? c.V - tb : kTile;
        bool closed[4] = {true, true, true, true};   // dn0 dn1 up0 up1
        for (int l = 0; l < kTile; l++) {
            const int i = tb + (l < nw ? l : nw - 1);
            if (i < 0 || i >= c.V || i - tb >= kTile) fail("lane", c, i);
            const Geo g = make_geo_inv(c, i);
            const int d[4] = {g.dn(0), g.dn(1), g.up(0), g.up(1)};
            for (int x = 0; x < 4; x++) closed[x] = closed[x] && (unsigned)(i + d[x] - tb) < (unsigned)nw;
        }
        for (int x = 0; x < 4; x++) {
            if (!closed[x]) continue;
            std::vector<int> read(kTile, 0);
            for (int l = 0; l < nw; l++) {
                checked++;
                const Geo g = make_geo_inv(c, tb + l);
                const int k = l + (x < 2 ? g.dn(x) : g.up(x - 2));
                if (k < 0 || k >= nw) fail("slot", c, tb + l);
                else read[k]++;
            }
            for (int l = 0; l < nw; l++)
                if (read[l] != 1) fail("slot read", c, tb + l);
        }
    }
}

static void columns(std::array<int, 4> d, int chunk) {
    CfgDesc c = desc(d);
    c.tchunk = chunk;
    const int n = (c.V + kTile - 1) / kTile;
    std::vector<int> seen(n, 0);
    for (int j = 0; j < n; j++) {
        checked++;
        const int t = tile_order(j, c);
        if (t < 0 || t >= n || seen[t]++) fail("tile order", c, j);
    }
}

// Launch orders: every block of a launch (padded to a multiple of eight) once,
// the padding past the end, whatever the number of blocks.
static void orders(int n) {
    std::vector<char> runs(n, 0), deal(n, 0);
    int live = 0, wrong = 0;
    for (int j = 0; j < n; j++) {
        const int t = run_order(j, n);
        if (t < 0 || t >= n || runs[t]++) wrong++;
    }
    for (int b = 0; b < (n + 7) / 8 * 8; b++) {
        const int t = deal_block(b, n, 1);
        if (t >= n) continue;
        live++;
        if (t < 0 || deal[t]++) wrong++;
    }
    checked += 2 * n;
    if (live != n || wrong) {
        std::fprintf(stderr, "violation: launch order of %d blocks\n", n);
        bad++;
    }
}

int main() {
    for (int n = 1; n < 200; n++) orders(n);
    for (int n : {8 * kDeal - 1, 8 * kDeal, 8 * kDeal + 1, 8 * kDeal + 7, 16 * kDeal + 13, 62400,
                  147456, 524287})
        orders(n);
    columns({16, 16, 48, 48}, 16);
    columns({32, 32, 96, 12}, 64);
    columns({20, 20, 60, 5}, 25);
    columns({24, 24, 72, 3}, 36);
    columns({8, 8, 24, 24}, 0);
    const std::vector<std::array<int, 4>> small = {
        {2, 2, 2, 2}, {4, 4, 12, 12}, {3, 5, 4, 7}, {8, 8, 24, 24}, {6, 6, 18, 18}, {10, 10, 6, 6},
        {7, 7, 21, 5}, {9, 9, 9, 9}, {16, 16, 8, 4}, {64, 2, 2, 2}, {2, 32, 3, 2}, {65, 3, 2, 2},
        {5, 3, 2, 13}, {2, 2, 31, 2}, {12, 12, 36, 4}, {32, 32, 4, 3}, {3, 21, 2, 2}, {21, 3, 5, 2}};
    for (auto &d : small) {
        const CfgDesc c = desc(d);
        for (int i = 0; i < c.V; i++) same(c, i);
        tiles(c);
    }
    const std::vector<std::array<int, 4>> big = {{2, 2, 2, 33554400}, {2, 2, 33554400, 2},
        {2, 33554400, 2, 2}, {33554400, 2, 2, 2}, {3, 3, 3, 9942043}, {8, 8, 1752, 1752},
        {7, 11, 13, 268000}, {127, 129, 127, 129}, {3, 9942043, 3, 3}};
    std::srand(1);
    for (auto &d : big) {
        const CfgDesc c = desc(d);
        const long long V = c.V;
        const long long step[3] = {d[0], 1LL * d[0] * d[1], 1LL * d[0] * d[1] * d[2]};
        for (long long s : step)
            for (int k = 0; k < 400000; k++) {
                const long long q = k < 1000 ? k : k < 2000 ? V / s - (k - 1000)
                                    : (1LL * std::rand() * RAND_MAX + std::rand()) % (V / s + 1);
                for (int x = -2; x <= 2; x++) {
                    const long long i = q * s + x;
                    if (i >= 0 && i < V) same(c, (int)i);
                }
            }
        for (int i = 0; i < 100000; i++) {
            same(c, i);
            same(c, c.V - 1 - i);
        }
    }
    std::printf("%lld checks, %lld violations\n", checked, bad);
    return bad ? 1 : 0;
}
