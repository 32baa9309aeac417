// Host check of the direct form's merge of neighbouring bits (or_runs of
// paper_2009_09500_amd/csrc/vox_direct.h): its lanes, modelled 16 at a time as
// the kernel takes a segment's samples, set exactly the segment's voxels in
// every volume in which the library's rule (direct_runs) lets it merge, up to
// the largest volumes a call may have, around 2^32 words.  No volume is held:
// the words that the model writes are kept in a map.  Built and run by
// tests/test_direct_runs.py (CPU only).
//
// argv[1] = "always": merge whatever the volume (a planted mistake that the
// check must see).  Prints the merged segments, those set bit by bit, and the
// segments whose words differ.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>

#include "vox_direct.h"

typedef std::map<uint64_t, uint32_t> Words;

// The lanes' row shifts: lane i of the result holds lane i - by's value (`out`
// where there is none; by = -1: the next lane's).
static uint32_t shifted(const uint32_t* v, int i, int by, uint32_t out) {
    return i - by >= 0 && i - by < 16 ? v[i - by] : out;
}

// One step of 16 samples with bit indexes b, of which the first `count` are the
// segment's (the others are whatever the lanes step to).
static void merge(const uint64_t b[16], int count, bool last, Words& out) {
    uint32_t word[16], bits[16];
    for (int i = 0; i < 16; ++i) {
        word[i] = (uint32_t)(b[i] >> 5);
        bits[i] = i < count ? 1u << (b[i] & 31u) : 0u;
    }
    for (int by = 1; by < 16; by *= 2) {
        uint32_t next[16];
        for (int i = 0; i < 16; ++i)
            next[i] = bits[i] | (shifted(word, i, by, ~word[i]) == word[i] ? shifted(bits, i, by, 0u) : 0u);
        memcpy(bits, next, sizeof(bits));
    }
    for (int i = 0; i < 16; ++i) {
        const bool in = i < count, end = last && i == count - 1;
        if (in && bits[i] != 0u && (end || shifted(word, i, -1, ~word[i]) != word[i])) out[b[i] >> 5] |= bits[i];
    }
}

int main(int argc, char** argv) {
    const bool always = argc > 1 && !strcmp(argv[1], "always");
    uint64_t merged = 0, single = 0, bad = 0, seed = 3;
    auto rnd = [&](int64_t n) {
        seed = seed * 6364136223846793005ull + 1442695040888963407ull;
        return (int64_t)((seed >> 20) % (uint64_t)n);
    };
    const int64_t volumes[][3] = {
        {300, 251, 199}, {1, 40, 30}, {3, 31, 17}, {33, 20, 40}, {1 << 20, 1 << 10, 3},
        // 2^32 words and more: slabs of 2^32, 2^31, 2^30 and 2^28 words.
        {1 << 19, 1 << 18, 2}, {1 << 20, 1 << 17, 2}, {1 << 18, 1 << 18, 4}, {1 << 17, 1 << 17, 16}, {1 << 18, 1 << 16, 16},
        {1 << 17, 1 << 17, 9}, {1 << 17, 1 << 17, 8}, {1 << 19, 1 << 18, 1}, {1 << 20, 1 << 14, 8}, {1 << 20, 1 << 14, 16},
        {1 << 16, 1 << 16, 32}, {1 << 16, 1 << 16, 33}, {1 << 16, 1 << 16, 64}};
    for (const auto& dim : volumes) {
        const int64_t nwords = (dim[0] * dim[1] * dim[2] + 31) / 32;
        const bool runs = always || vox::direct_runs(vox::kRunsMinSegments + 1, nwords);
        for (int s = 0; s < 4000; ++s) {
            // Steep segments of up to 100 steps, from corners or anywhere.
            int64_t p0[3], d[3], n = 0;
            for (int a = 0; a < 3; ++a) {
                const int64_t reach = dim[a] < 100 ? dim[a] : (s % 3 == 0 ? 4 : 100);
                int64_t p1;
                p0[a] = s % 2 ? rnd(dim[a]) : rnd(reach);
                p1 = p0[a] + rnd(2 * reach + 1) - reach;
                p1 = p1 < 0 ? 0 : (p1 >= dim[a] ? dim[a] - 1 : p1);
                d[a] = p1 - p0[a];
                n = std::llabs(d[a]) > n ? std::llabs(d[a]) : n;
            }
            Words expect, got;
            for (int64_t c0 = 0; c0 <= n; c0 += 16) {
                uint64_t b[16];
                for (int64_t i = 0; i < 16; ++i) {
                    int64_t v[3];
                    for (int a = 0; a < 3; ++a) {
                        const int64_t num = 2 * (c0 + i) * d[a] + n, den = n ? 2 * n : 1;
                        v[a] = p0[a] + (num >= 0 ? num / den : -((-num + den - 1) / den));
                    }
                    b[i] = (uint64_t)((v[2] * dim[1] + v[1]) * dim[0] + v[0]);
                    if (c0 + i <= n) expect[b[i] >> 5] |= 1u << (b[i] & 31u);
                }
                const int count = n - c0 < 15 ? (int)(n - c0) + 1 : 16;
                if (runs) {
                    merge(b, count, c0 + 16 > n, got);
                } else {
                    for (int i = 0; i < count; ++i) got[b[i] >> 5] |= 1u << (b[i] & 31u);
                }
            }
            ++(runs ? merged : single);
            if (got != expect) ++bad;
        }
    }
    printf("merged %llu single %llu bad %llu\n", (unsigned long long)merged, (unsigned long long)single,
           (unsigned long long)bad);
    return bad != 0;
}
