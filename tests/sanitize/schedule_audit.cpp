// Host audit of the stage launches' shapes and orders (test infrastructure),
// with the runtime's own rules (schedule.h): the column width that tile_chunk
// gives a box divides its slice's tiles, and with it tile_order visits every
// tile once; the same for the LDS-staged blocks (block_chunk, block_order); the
// default kernel's rule.
#include <hip/hip_runtime.h>

#include <array>
#include <cstdio>
#include <set>
#include <vector>

#include "lattice_dev.h"
#include "layout.h"
#include "schedule.h"

using namespace tgf;

static long long checked = 0, bad = 0;
static void fail(const char *what, const int d[4]) {
    if (bad < 20) std::fprintf(stderr, "violation: %s %dx%dx%dx%d\n", what, d[0], d[1], d[2], d[3]);
    bad++;
}

static std::set<int> widths;

static void orders(std::array<int, 4> a) {
    const int *d = a.data();
    CfgDesc c{};
    c.V = 1;
    for (int m = 0; m < 4; m++) {
        c.d[m] = d[m];
        c.V *= d[m];
    }
    const int slice_sites = d[0] * d[1] * d[2];
    c.tchunk = tile_chunk(d);
    widths.insert(c.tchunk);
    checked++;
    if (c.tchunk && (slice_sites % kTile || (slice_sites / kTile) % c.tchunk ||
                     slice_sites / kTile <= kTileSlice))
        fail("tile columns", d);
    const int nt = (c.V + kTile - 1) / kTile;
    std::vector<char> seen(nt, 0);
    for (int j = 0; j < nt; j++) {
        checked++;
        const int t = tile_order(j, c);
        if (t < 0 || t >= nt || seen[t]++) fail("tile order", d);
    }
    c.blk = default_block(d);
    c.chunk = block_chunk(d, c.blk);
    if (c.blk < 64 || c.blk > kBlock) fail("block", d);
    if (c.chunk && (slice_sites % c.blk || (slice_sites / c.blk) % c.chunk)) fail("block columns", d);
    const int nb = (c.V + c.blk - 1) / c.blk;
    std::vector<char> seen_b(nb, 0);
    for (int j = 0; j < nb; j++) {
        checked++;
        const int t = block_order(j, c);
        if (t < 0 || t >= nb || seen_b[t]++) fail("block order", d);
    }
}

// The default kernel is a rule of extents and storage; both answers on each
// side of its lines.
static void defaults() {
    struct Want { std::array<int, 4> d; bool f64, f32, c12; };
    for (const Want &w : std::vector<Want>{
             {{8, 8, 24, 24}, false, false, false},     {{9, 9, 27, 27}, false, false, false},
             {{9, 9, 54, 54}, false, false, false},     {{9, 9, 81, 81}, false, true, false},
             {{9, 9, 162, 162}, false, true, true},     {{9, 9, 324, 324}, true, true, true},
             {{8, 8, 384, 384}, false, false, false},   {{12, 12, 256, 256}, false, false, false},
             {{16, 16, 48, 48}, false, false, false},   {{16, 16, 192, 192}, true, true, false},
             {{32, 32, 96, 96}, true, true, false},     {{36, 36, 108, 108}, false, false, false},
             {{64, 64, 48, 48}, false, false, false},   {{6, 6, 252, 252}, false, true, true},
             {{2, 2, 8192, 8190}, false, false, false}}) {
        checked += 3;
        if (lds_by_default(w.d.data(), true, false) != w.f64 ||
            lds_by_default(w.d.data(), false, false) != w.f32 ||
            lds_by_default(w.d.data(), false, true) != w.c12)
            fail("default kernel", w.d.data());
    }
}

int main() {
    defaults();
    for (int l = 2; l <= 40; l++) orders({l, l, 3 * l, 3});
    for (int l : {2, 3, 5, 8, 16, 20, 24, 31, 32, 64})
        for (int m : {2, 7, 16, 32, 48})
            for (int n : {2, 5, 72, 96, 192, 257}) orders({l, m, n, 2});
    orders({16, 16, 72, 4});
    orders({128, 128, 16, 5});
    // the rule is in use: site order, and columns of several widths
    checked++;
    if (!widths.count(0) || widths.size() < 4) {
        std::fprintf(stderr, "violation: only %zu column widths\n", widths.size());
        bad++;
    }
    std::printf("%lld checks, %lld violations\n", checked, bad);
    return bad ? 1 : 0;
}
