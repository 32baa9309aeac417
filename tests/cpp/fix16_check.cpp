// Host check of the 16.16 coordinates of the int16 lists (fix30_slope,
// fix16_* of paper_2009_09500_amd/csrc/vox_device.h, the library's own code
// built for the host) against eq. (3)'s integer divisions: every N up to
// kFix16MaxN (or argv[1]), slopes near 0, 1/2 and 1 and any, both signs, from
// start voxels anywhere, `steps` voxels from each.  argv[2]: steps (7, a
// lane's); more of them, or longer segments, must fail somewhere.
// Built and run by tests/test_fix16.py (CPU only).
#include <cstdio>
#include <cstdlib>

#include "vox_device.h"

int main(int argc, char** argv) {
    const uint32_t n_max = argc > 1 ? (uint32_t)atoi(argv[1]) : vox::kFix16MaxN;
    const uint32_t steps = argc > 2 ? (uint32_t)atoi(argv[2]) : 7u;
    uint64_t cases = 0, bad = 0, seed = 7;
    auto rnd = [&](uint32_t n) {
        seed = seed * 6364136223846793005ull + 1442695040888963407ull;
        return (uint32_t)((seed >> 33) % n);
    };
    for (uint32_t n = 1; n <= n_max; ++n) {
        const double rcp = 1.0 / (double)n;
        for (int i = 0; i < 40; ++i) {
            uint32_t a = i < 4 ? (uint32_t)i : i < 8 ? n - (uint32_t)(i - 4) : i < 12 ? n / 2 + (uint32_t)(i - 10)
                                                                                      : rnd(n + 1);
            if (a > n) a = n;
            const int32_t d = (i & 1) ? -(int32_t)a : (int32_t)a;
            int32_t p0 = (int32_t)rnd(65536) - 32768;
            if (i == 20) p0 = d < 0 ? 32767 : -32768;
            if (p0 + d > 32767) p0 = 32767 - d;
            if (p0 + d < -32768) p0 = -32768 - d;
            const int32_t point = vox::fix16_point(p0), slope = vox::fix30_slope(d, rcp);
            const int32_t step = vox::fix16_step(slope);
            for (int t = 0; t < 8; ++t) {
                const uint32_t k0 = t == 0 ? 0u : t == 1 ? n : rnd(n + 1);
                int32_t v = vox::fix16_at(point, slope, k0);
                for (uint32_t k = k0; k <= n && k <= k0 + steps; ++k, v = (int32_t)((uint32_t)v + (uint32_t)step)) {
                    const int64_t num = 2ll * k * d + n, den = 2ll * n;
                    const int64_t q = num >= 0 ? num / den : -((-num + den - 1) / den);
                    ++cases;
                    if ((v >> 16) != p0 + q) ++bad;
                }
            }
        }
    }
    printf("cases %llu bad %llu\n", (unsigned long long)cases, (unsigned long long)bad);
    return bad != 0;
}
