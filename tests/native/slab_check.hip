// Host check of the slab order (lattices without whole-tile z-groups): the
// blocks of a launch visit every tile of a half lattice exactly once, the
// rest of them get the tile after the last one, the pad is less than one
// tile per slab and slice on average plus one, and every XCD's share differs
// by at most one tile per slice.  Prints "cases N bad B".
#include "lqcd_internal.h"
#include "hop_common.h"

#include <cstdio>
#include <vector>

using namespace lqcd;

int main() {
    int bad = 0, cases = 0, slabs = 0;
    const int L[][4] = {{18, 18, 42, 40}, {28, 28, 28, 28}, {26, 26, 26, 40}, {22, 20, 36, 36},
                        {46, 46, 46, 50}, {30, 30, 30, 30}, {62, 58, 16, 10}, {34, 18, 18, 54},
                        {2, 2, 256, 512}, {6, 258, 18, 20}, {18, 18, 18, 1024}};
    for (const auto &d : L) {
        ++cases;
        Geom g{};
        for (int m = 0; m < 4; ++m) g.L[m] = d[m];
        g.lxh = d[0] / 2;
        g.sy = g.lxh;
        g.sz = g.sy * d[1];
        g.st = g.sz * d[2];
        g.vh = g.st * d[3];
        g.ntiles = (g.vh + TILE - 1) / TILE;
        if (!use_slabs(g, brick_plan(g, LQCD_F64, 0), true)) continue;
        ++slabs;
        const Brick k = make_slab_brick(g);
        const int64_t n = brick_blocks(g, k);
        std::vector<int> seen(g.ntiles + 1, 0);
        int64_t share[8] = {};
        bool ok = n % 8 == 0 && n < ((int64_t)1 << 31);
        for (int64_t b = 0; b < n && ok; ++b) {
            const int64_t t = brick_order((uint32_t)b, k, g);
            if (t < 0 || t > g.ntiles) ok = false;
            else {
                seen[t] += 1;
                if (t < g.ntiles) share[b / (n / 8)] += 1;
            }
        }
        for (int64_t t = 0; t < g.ntiles; ++t) ok = ok && seen[t] == 1;
        for (int x = 0; x < 8; ++x) ok = ok && 8 * share[x] <= g.ntiles + 8 * (int64_t)g.L[3] && 8 * share[x] >= g.ntiles - 8 * (int64_t)g.L[3];
        ok = ok && n - g.ntiles <= 2 * 8 * (int64_t)g.L[3];
        if (!ok) {
            ++bad;
            printf("FAIL %dx%dx%dx%d\n", d[0], d[1], d[2], d[3]);
        }
    }
    printf("cases %d slabs %d bad %d\n", cases, slabs, bad);
    return bad ? 1 : 0;
}
