// Host check of how small bit-volume calls deal words to workgroups
// (paper_2009_09500_amd/csrc/vox_slabs.h, the library's own code built for the
// host): whatever the estimated work of the runs, the cut covers every word
// once, in multiples of 32 words, no workgroup gets more than the room it has,
// and where the cut is by work a run that does all of it is shared by an eighth
// of the workgroups at least.  Built and run by tests/test_slab_cut.py (CPU
// only).
//
// argv[1] = "light": the words weigh a sixth of what they do (a planted mistake
// that the check must see).  Prints the cuts by work and by words alone, and the
// faults.
#include <cstdio>
#include <cstring>
#include <vector>

#include "vox_slabs.h"

int main(int argc, char** argv) {
    const bool light = argc > 1 && !strcmp(argv[1], "light");
    uint64_t cuts = 0, even = 0, bad = 0, seed = 11;
    auto rnd = [&](uint64_t n) {
        seed = seed * 6364136223846793005ull + 1442695040888963407ull;
        return (uint32_t)((seed >> 24) % n);
    };
    for (uint32_t words = 64; words <= 16384; words = words < 256 ? words + 32 : (words + words / 5) / 32 * 32) {
        for (uint32_t trial = 0; trial < 600; ++trial) {
            const uint32_t runs = trial % 7 == 0 ? 1 + rnd(8) : (trial % 3 ? 256 : 1 + rnd(vox::kSlabMaxRuns));
            const uint32_t nwords = (runs - 1) * words + 1 + rnd(words);
            const uint32_t samples = trial % 5 ? vox::kSlabSamples : 1 + rnd(vox::kSlabSamples), n = samples * (1 + rnd(32));
            // Samples over all runs, in some of them, or in one.
            std::vector<uint32_t> load(runs, 0u);
            const uint32_t width = trial % 4 == 0 ? runs : 1 + rnd(trial % 4 == 1 ? 1 : runs), from = rnd(runs - width + 1);
            const uint32_t longest = 1 + rnd(trial % 11 ? 3000 : 1 << 20);
            for (uint32_t s = 0; s < samples; ++s) {
                const bool astray = trial % 2 && rnd(10) == 0;
                uint32_t a = astray ? rnd(runs) : from + rnd(width), b = astray ? rnd(runs) : from + rnd(width);
                if (a > b) std::swap(a, b);
                const uint32_t work = vox::slab_work(rnd(longest), b - a + 1u);
                for (uint32_t r = a; r <= b; ++r) load[r] += work;
            }
            uint64_t sum = 0;
            uint32_t max = 0;
            for (uint32_t w : load) {
                sum += w;
                max = w > max ? w : max;
            }
            if (sum >> 32) ++bad;
            if (!vox::slab_uneven((uint32_t)sum, max, runs, n, samples, words)) {
                ++even;
                continue;
            }
            ++cuts;
            // (Segments of less than `longest` steps.)
            if (!vox::slab_look(n, (int32_t)longest, words)) ++bad;
            const uint32_t base = vox::slab_base((uint32_t)sum, runs) / (light ? 6u : 1u);
            if ((uint64_t)base * runs + sum >= 1ull << 32) ++bad;
            const uint32_t total = base * runs + (uint32_t)sum;
            uint32_t at = 0, most = 0;
            std::vector<uint32_t> share(runs, 0u);  // workgroups with words of each run
            for (uint32_t r = 1; r <= runs; ++r) {
                uint32_t next = nwords;
                if (r < runs) {
                    const uint32_t target = vox::slab_target(r, runs, total);
                    uint32_t i = 0, before = 0;
                    while (i + 1 < runs && before + base + load[i] <= target) before += base + load[i++];
                    next = vox::slab_word(target, i, before, base + load[i], words, nwords);
                    if (next % 32u != 0u) ++bad;
                }
                if (next < at || next > nwords) ++bad;
                if (next - at > vox::slab_room(words)) ++bad;
                for (uint32_t i = at / words; at < next && i <= (next - 1) / words; ++i) ++share[i];
                at = next;
            }
            if (at != nwords) ++bad;
            for (uint32_t i = 0; i < runs; ++i)
                if (load[i] == max) most = share[i] > most ? share[i] : most;
            // (As many shares as the run has of 32 words, at most.)
            if (max == sum && runs >= 64 && most < (runs / 8 < words / 64 ? runs / 8 : words / 64)) ++bad;
        }
    }
    printf("cuts %llu even %llu bad %llu\n", (unsigned long long)cuts, (unsigned long long)even, (unsigned long long)bad);
    return bad != 0;
}
