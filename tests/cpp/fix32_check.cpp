// Host check of the 32-bit fractions that step an axis under the Euclidean N
// (fix32_* of paper_2009_09500_amd/csrc/vox_device.h, the library's own code built
// for the host) against eq. (3)'s integer divisions, for every kind of axis a <= N
// and both signs:
//   walk   whole walks from a remainder at any sample (counts of the lists)
//   list   quotient and fraction at any sample, and the steps from there (voxels of
//          the lists), also an axis with a = N
//   piece  chunks of 32 samples from a float reciprocal off by -1, 0 and +1 ulp
// argv[1]: the form.  argv[2]: the longest N.  argv[3], a planted mistake that the
// check must see: "floor" (rounded down), "unsigned" (list: no start of its own for a
// negative axis), "steps" (piece: chunks of 64).
// Prints the number of (N, a, k) cases and of differing steps.  Built and run by
// tests/test_fix32.py (CPU only).
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "vox_device.h"

int main(int argc, char** argv) {
    const char* form = argv[1];
    const uint32_t n_max = (uint32_t)atoi(argv[2]);
    const char* plant = argc > 3 ? argv[3] : "";
    const bool down = !strcmp(plant, "floor"), one_start = !strcmp(plant, "unsigned");
    const uint32_t chunk = !strcmp(plant, "steps") ? 64u : 32u;
    uint64_t cases = 0, bad = 0, seed = 5;
    auto rnd = [&](uint32_t n) {
        seed = seed * 6364136223846793005ull + 1442695040888963407ull;
        return (uint32_t)((seed >> 33) % n);
    };
    // All short lengths, some of the others, and the longest.
    for (uint32_t n = 1; n <= n_max; n += n < 200 ? 1 : n + 60 > n_max ? 1 : 1 + rnd(n_max / 40)) {
        const uint32_t two_n = 2u * n;
        for (int i = 0; i < 40; ++i) {
            const uint32_t a = i < 6 ? std::min<uint32_t>(i, n) : i < 12 ? n - std::min<uint32_t>(i - 6, n)
                               : i < 16 ? std::min<uint32_t>(n / 2 + (i - 13), n) : rnd(n + 1);
            const uint32_t neg = i & 1u;
            // Samples: all of the segment, from the start or on the way.
            const uint32_t k0 = i % 3 == 0 ? 0u : rnd(n + 1);
            auto num = [&](uint32_t k) { return 2ull * k * a + n - neg; };
            const uint32_t r = (uint32_t)(num(k0) % two_n);
            if (!strcmp(form, "walk")) {
                if (a == n) continue;  // (counted without a walk)
                const double unit = 0x1p32 / (double)two_n;
                uint32_t f = vox::fix32_of(r, unit), d = vox::fix32_of(2u * a, unit);
                if (down) f = (uint32_t)(r * unit), d = (uint32_t)(2u * a * unit);
                ++cases;
                for (uint32_t k = k0; k < n; ++k) {
                    const bool moved = num(k + 1) / two_n != num(k) / two_n;
                    if (__builtin_uadd_overflow(f, d, &f) != moved) ++bad;
                }
            } else if (!strcmp(form, "list")) {
                const double rcp_n = 1.0 / (double)n;
                uint32_t d = vox::fix32_slope(a, n, rcp_n);
                if (down && a != n) d = (uint32_t)((double)a * 0x1p32 * rcp_n);
                const uint32_t start = one_start ? 0x80000000u : vox::fix32_start(rcp_n);
                const uint64_t at = vox::fix32_at(k0, d, neg != 0, start);
                uint32_t f = (uint32_t)at;
                ++cases;
                if (at >> 32 != num(k0) / two_n) ++bad;
                // (The step to a sample has carried exactly when its fraction is below the slope.)
                if (k0 > 0 && (f < d) != (num(k0) / two_n != num(k0 - 1) / two_n)) ++bad;
                for (uint32_t k = k0; k < n; ++k) {
                    const bool moved = num(k + 1) / two_n != num(k) / two_n;
                    if (__builtin_uadd_overflow(f, d, &f) != moved) ++bad;
                }
            } else {
                if (a == n) continue;  // (moves at every step, without fractions)
                const float exact = 1.0f / (float)two_n;
                for (float rcp : {std::nextafterf(exact, 0.0f), exact, std::nextafterf(exact, 2.0f)}) {
                    const float scale = rcp * 0x1p32f;
                    uint32_t f = vox::fix32_about(r, scale), d = vox::fix32_about(2u * a, scale);
                    if (down) f -= 2048u + 1024u, d -= 2048u + 1024u;
                    ++cases;
                    for (uint32_t k = k0; k < n && k + 1 < k0 + chunk; ++k) {
                        const bool moved = num(k + 1) / two_n != num(k) / two_n;
                        if (__builtin_uadd_overflow(f, d, &f) != moved) ++bad;
                    }
                }
            }
        }
    }
    printf("cases %llu bad %llu\n", (unsigned long long)cases, (unsigned long long)bad);
    return bad != 0;
}
