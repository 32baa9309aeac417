// Host check of the 16.16 coordinates of the int16 lists (fix30_slope, fix16_* of
// paper_2009_09500_amd/csrc/vox_device.h, the library's own code built for the host)
// against eq. (3)'s integer divisions: for the lengths given, every slope of both
// signs, from every voxel, and seven voxels from each.  Built and run by
// tests/test_fix16_slopes.py (CPU only).  Prints the number of voxels and of
// differing ones.
#include <cstdio>
#include <cstdlib>

#include "vox_device.h"

int main(int argc, char** argv) {
    uint64_t cases = 0, bad = 0;
    for (int arg = 1; arg < argc; ++arg) {
        const int32_t n = atoi(argv[arg]);
        const double rcp = 1.0 / (double)n;
        for (int32_t d = -n; d <= n; ++d) {
            const int32_t p0 = d < 0 ? 32767 : -32768;
            const int32_t point = vox::fix16_point(p0), slope = vox::fix30_slope(d, rcp), step = vox::fix16_step(slope);
            // Voxel 2 k d + n over 2 n, stepped exactly.
            int32_t q = 0, r = n;
            for (int32_t k0 = 0; k0 <= n; ++k0) {
                int32_t v = vox::fix16_at(point, slope, (uint32_t)k0), qq = q, rr = r;
                for (int32_t k = k0; k <= n && k <= k0 + 7; ++k, v = (int32_t)((uint32_t)v + (uint32_t)step)) {
                    ++cases;
                    if ((v >> 16) != p0 + qq) ++bad;
                    rr += 2 * d;
                    if (rr >= 2 * n) rr -= 2 * n, ++qq;
                    if (rr < 0) rr += 2 * n, --qq;
                }
                r += 2 * d;
                if (r >= 2 * n) r -= 2 * n, ++q;
                if (r < 0) r += 2 * n, --q;
            }
        }
    }
    printf("cases %llu bad %llu\n", (unsigned long long)cases, (unsigned long long)bad);
    return bad != 0;
}
