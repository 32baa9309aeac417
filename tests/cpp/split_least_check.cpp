// Host check of how many records a part of a cut brick has at least (split_least
// of paper_2009_09500_amd/csrc/vox_exact.h): within [kSplitLeast, kSplitMost], fewer
// for longer pieces, more where the parts' flushes cost more, and for no sample
// kSplitMost.  With any of them the extra items stay within their tables.  Built
// and run by tests/test_split_least.py (CPU only).  Prints "ok" or the first
// failure.
#include <cstdio>
#include <random>

#include "vox_exact.h"

int main() {
    std::mt19937_64 rng(7);
    auto log_up_to = [&](double most) { return (uint64_t)std::exp(std::uniform_real_distribution<>(0.0, std::log(most))(rng)); };
    for (int trial = 0; trial < 200000; ++trial) {
        const uint64_t total = log_up_to(4294967294.0), words = log_up_to(1e18);
        const uint32_t pieces = (uint32_t)log_up_to(200000.0), busy = (uint32_t)(rng() % (vox::kSplitFewBricks + 1u));
        const uint32_t voxels = (uint32_t)(rng() % 50u == 0 ? 0u : log_up_to(4.2e6));
        const uint32_t t = vox::split_least(total, voxels, pieces, words, busy);
        const uint32_t longer = vox::split_least(total, voxels * 2u, pieces, words, busy);
        const uint32_t wider = vox::split_least(total, voxels, pieces, words * 4u, busy);
        if (t < vox::kSplitLeast || t > vox::kSplitMost || longer > t || wider < t ||
            ((voxels == 0u || busy == 0u) && t != vox::kSplitMost)) {
            printf("total %llu voxels %u pieces %u words %llu busy %u: %u, longer %u, wider %u\n", (unsigned long long)total,
                   voxels, pieces, (unsigned long long)words, busy, t, longer, wider);
            return 1;
        }
        // One brick with all records makes the most items.
        const uint64_t T = vox::split_threshold(total, t);
        if (vox::brick_items((uint32_t)total, T) - 1u > vox::kMaxExtraItems) {
            printf("total %llu: %u items of %llu\n", (unsigned long long)total, vox::brick_items((uint32_t)total, T),
                   (unsigned long long)T);
            return 1;
        }
    }
    printf("ok\n");
    return 0;
}
