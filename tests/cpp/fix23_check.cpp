// Host check of the 23-bit fractions that step a piece's minor axes (fix23_*
// of paper_2009_09500_amd/csrc/vox_device.h, the library's own code built for
// the host): with the reciprocal off by -1, 0 and +1 ulp, the quotients they
// give over a piece equal eq. (3)'s integer divisions.  Built and run by
// tests/test_fix23.py (CPU only).
//
// argv[1]: samples of a piece (256: the longest); argv[2] = "floor": slopes
// rounded down (a planted mistake the check must see).
// Prints the number of (N, a, r) cases and of mismatching quotients.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "vox_device.h"

int main(int argc, char** argv) {
    const uint32_t len = argc > 1 ? (uint32_t)atoi(argv[1]) : 256u;
    const bool floor_slope = argc > 2 && !strcmp(argv[2], "floor");
    uint64_t cases = 0, bad = 0, seed = 1;
    auto rnd = [&](uint32_t n) {
        seed = seed * 6364136223846793005ull + 1442695040888963407ull;
        return (uint32_t)((seed >> 33) % n);
    };
    for (uint32_t n = 1; n <= 16384; n += n < 300 ? 1 : 1 + rnd(40)) {
        const uint32_t two_n = 2u * n;
        const float exact = 1.0f / (float)two_n;
        const float rcps[3] = {std::nextafterf(exact, 0.0f), exact, std::nextafterf(exact, 2.0f)};
        for (int i = 0; i < 48; ++i) {
            // Slopes near 0, near 1, the tie, and any.
            const uint32_t a = i < 4 ? std::min<uint32_t>(i, n) : i < 8 ? n - std::min<uint32_t>(i - 4, n) : rnd(n + 1);
            // Remainders a piece can start with: (2 k a + n - neg) mod 2n.
            const uint32_t neg = i & 1u;
            const uint32_t k = i < 16 ? 0u : rnd(n + 1);
            const uint64_t num0 = 2ull * k * a + n - neg;
            const uint32_t r = (uint32_t)(num0 % two_n);
            for (float rcp : rcps) {
                const uint32_t f = vox::fix23_fraction(r, 2u * a, two_n, rcp);
                uint32_t s = vox::fix23_slope(2u * a, two_n, rcp);
                if (floor_slope && a < n) s = (uint32_t)(((uint64_t)a << 23) / n);
                ++cases;
                if (f >> 23 || s >> 23) ++bad;
                const uint32_t steps = std::min<uint32_t>(len, n - k + 1);
                for (uint32_t j = 0; j < steps; ++j) {
                    // As the fill starts a chunk at j, and as it steps: the
                    // same integers, since both are f + j s.
                    const uint64_t t = (uint64_t)f + (uint64_t)j * s;
                    if (t >= (1ull << 31) || t >> 23 != ((uint64_t)r + 2ull * j * a) / two_n) ++bad;
                }
            }
        }
    }
    printf("cases %llu bad %llu\n", (unsigned long long)cases, (unsigned long long)bad);
    return bad != 0;
}
