// Host check of the slab order's plan (csrc/hop_common.h): the most tiles of a
// slab in one slice, which the launch takes from a closed form, against a
// count over all slabs and slices; and that the pads of the order never put a
// launch of 512 threads per block beyond the 2^32 work items that one counts.
// Prints "cases N bad B".
#include "lqcd_internal.h"
#include "hop_common.h"

#include <cstdio>

using namespace lqcd;

int main() {
    int cases = 0, bad = 0;
    auto geom = [](int x, int y, int z, int t) {
        Geom g{};
        g.L[0] = x, g.L[1] = y, g.L[2] = z, g.L[3] = t;
        g.lxh = x / 2;
        g.sy = g.lxh;
        g.sz = g.sy * y;
        g.st = g.sz * z;
        g.vh = g.st * t;
        g.ntiles = (g.vh + TILE - 1) / TILE;
        return g;
    };
    auto one = [&](const Geom &g) {
        uint32_t most = 1;
        for (uint32_t t = 0; t < (uint32_t)g.L[3]; ++t)
            for (uint32_t j = 0; j < 8; ++j) {
                const uint32_t n = slab_tile(g, t, j + 1) - slab_tile(g, t, j);
                if (n > most) most = n;
            }
        const Brick k = make_slab_brick(g);
        ++cases;
        if (k.pt.d != most || k.ptg != most) {
            ++bad;
            printf("FAIL %dx%dx%dx%d: %u, counted %u\n", g.L[0], g.L[1], g.L[2], g.L[3], k.pt.d, most);
        }
    };
    for (int x = 2; x <= 62; x += 4)
        for (int y = 2; y <= 62; y += 4)
            for (int z = 2; z <= 66; z += 2)
                for (int t : {2, 6, 34, 128}) {
                    const Geom g = geom(x, y, z, t);
                    if (g.st >= 8 * 8 * TILE) one(g);
                }
    // slices of 512 m + 4 sites, where two lengths of runs differ in tiles
    for (int m = 8; m < 1200; ++m)
        for (int y = 2; y <= 64; y += 2) {
            const int rest = (512 * m + 4) / (2 * y);
            if ((512 * m + 4) % (2 * y) == 0) one(geom(2 * rest, y, 2, 40));
        }
    for (int t = 1000; t <= 65536; t += t < 60000 ? 1000 : 14)
        for (int x : {82, 86, 94, 98, 102})
            for (bool both : {false, true}) {
                const Geom g = geom(x, 10, 10, t);
                const int64_t plain = g.ntiles * (both ? 2 : 1) * 512;
                if (plain > UINT32_MAX) continue;
                const Brick k = launch_brick(g, LQCD_F32, both ? 2 : 0, both);
                ++cases;
                if (brick_blocks(g, k) * (both ? 2 : 1) * 512 > UINT32_MAX) {
                    ++bad;
                    printf("FAIL %dx10x10x%d: %lld work items, %lld in plain order\n", x, t,
                           (long long)(brick_blocks(g, k) * (both ? 2 : 1) * 512), (long long)plain);
                }
            }
    printf("cases %d bad %d\n", cases, bad);
    return bad ? 1 : 0;
}
