// The direct form of the bit-volume output: every voxel ORed into its grid
// word with a device-scope atomic.  Correct for any volume shape; shared by
// the plain direct path (vox_grid.hip) and the scenes of a batch that the
// brick path does not serve (vox_brick.hip).
#pragma once

#include <type_traits>

#include "vox_device.h"
#include "vox_internal.h"

namespace vox {

// ORs the bits of neighbouring lanes of 16 with the same word together; true in
// the last lane of each such run, which then holds them.  `in`: the lane has a
// sample (the segment's first lanes do), `end`: its last one.  (A sample may hold
// no bit of its own.)  Atomics bound the direct form, about 25 G a
// second, and a segment along x sets up to 16 neighbouring bits: 50 000 uniform
// segments in 300x251x199 0.203 ms against 0.251, 16 384 in 960^3 0.312 / 0.345.
// Few segments are bound by the latency of their waves instead (log-uniform
// lengths in 960^3: 1000 0.0162 / 0.0122, 8000 0.0371 / 0.0364, 16 000 0.0619 /
// 0.0633), so fewer than kRunsMinSegments set bit by bit.  So do volumes of
// more than kRunsMaxWords words, whose samples can lie a multiple of 2^32 words
// apart (in 2^19 x 2^18 x 2 one z step does), for words are told apart by the low
// halves of their indexes.
constexpr int64_t kRunsMinSegments = 8192;
constexpr int64_t kRunsMaxWords = int64_t(1) << 32;
inline bool direct_runs(int64_t n, int64_t nwords) { return n > kRunsMinSegments && nwords <= kRunsMaxWords; }
__device__ __forceinline__ bool or_runs(uint32_t word, bool in, bool end, uint32_t& bits) {
    static_assert(kSampleLanes == 16, "one DPP row a segment");
    auto step = [&](auto shift) {
        constexpr int kDpp = 0x110 + decltype(shift)::value;  // row_shr
        const uint32_t w = (uint32_t)__builtin_amdgcn_update_dpp((int)~word, (int)word, kDpp, 0xf, 0xf, false);
        const uint32_t m = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)bits, kDpp, 0xf, 0xf, true);
        bits |= w == word ? m : 0u;
    };
    step(std::integral_constant<int, 1>{});
    step(std::integral_constant<int, 2>{});
    step(std::integral_constant<int, 4>{});
    step(std::integral_constant<int, 8>{});
    // (row_shl by one; the row's last lane has no next.)
    const uint32_t next = (uint32_t)__builtin_amdgcn_update_dpp((int)~word, (int)word, 0x101, 0xf, 0xf, false);
    return in && bits != 0u && (end || next != word);
}

// Segments [0, n) of one volume, four per wave, 16 lanes each; the waves of
// the launch take segment groups wave0, wave0 + wave_stride, ...  A
// segment's lanes take its samples 16 at a time (SampleAt), and each lane
// whose sample starts a new voxel ORs that voxel's bit into the grid.  Range
// check first: a segment with an end point outside the volume sets the
// status and writes nothing.  Counts: N + 1 for the Chebyshev N (also for a
// segment outside the volume), the number of voxels after duplicate removal
// for the Euclidean N of eq. (1) (0 outside the volume).
template <bool kAligned8, bool kEuclid, bool kRuns = false>
__device__ __forceinline__ void direct_segments(const int32_t* __restrict__ segs, int64_t n, int32_t dx,
                                                int32_t dy, int32_t dz, uint32_t* __restrict__ grid,
                                                int32_t* __restrict__ counts, int32_t* __restrict__ status,
                                                int64_t wave0, int64_t wave_stride) {
    constexpr int kSlots = kWave / kSampleLanes;
    const uint32_t lane = threadIdx.x % kWave;
    const uint32_t sub = lane % kSampleLanes;
    const uint32_t slot = lane / kSampleLanes;
    const uint64_t slot_bits = ((1ull << kSampleLanes) - 1) << (kSampleLanes * slot);
    const int32_t dim[3] = {dx, dy, dz};
    for (int64_t i0 = wave0 * kSlots; i0 < n; i0 += wave_stride * kSlots) {
        const int64_t i = i0 + slot;
        const bool valid = i < n;
        Seg g = {};
        if (valid) g = load_seg<kAligned8>(segs, i);
        bool ok = valid;
#pragma unroll
        for (int a = 0; a < 3; ++a)
            ok &= (g.p0[a] >= 0) & (g.p0[a] < dim[a]) & (g.p1[a] >= 0) & (g.p1[a] < dim[a]);
        if (valid && sub == 0) {
            if (!kEuclid && counts) {
                const int64_t N64 = seg_length(g);
                counts[i] = (int32_t)(N64 + 1 > 0x7FFFFFFFll ? 0x7FFFFFFFll : N64 + 1);
            }
            if (!ok) {
                if (kEuclid && counts) counts[i] = 0;
                atomicOr(status, kStatusOutOfRange);
            }
        }
        if (!ok) g = Seg{};
        // Inside the volume every side is below 2^20: N < 2^21.
        SampleAt s;
        s.init(g, kEuclid ? euclid_length(g) : (uint32_t)seg_length(g));
        bool moved = s.start(sub);
        uint32_t kept = 0;
        for (uint32_t c0 = 0; __ballot(ok && c0 <= s.N) != 0; c0 += kSampleLanes) {
            if (c0 != 0) moved = s.next();
            const bool in = ok && c0 + sub <= s.N, keep = moved && in;
            auto bit = [&] {
                return ((uint64_t)s.coord(g, 2) * (uint64_t)dy + (uint64_t)s.coord(g, 1)) * (uint64_t)dx +
                       (uint64_t)s.coord(g, 0);
            };
            if constexpr (kRuns) {
                const uint64_t b = bit();
                uint32_t bits = keep ? 1u << (uint32_t)(b & 31u) : 0u;
                if (or_runs((uint32_t)(b >> 5), in, c0 + sub == s.N, bits)) atomicOr(grid + (b >> 5), bits);
            } else if (keep) {
                const uint64_t b = bit();
                atomicOr(grid + (b >> 5), 1u << (uint32_t)(b & 31u));
            }
            if (kEuclid) kept += (uint32_t)__popcll(__ballot(keep) & slot_bits);
        }
        if (kEuclid && ok && sub == 0 && counts) counts[i] = (int32_t)kept;
    }
}

// Zeroes words [0, nwords) of a 16-byte-aligned volume; the threads of the
// launch take 16-byte units t0, t0 + t_stride, ...
__device__ __forceinline__ void clear_words(uint32_t* __restrict__ grid, int64_t nwords, int64_t t0,
                                            int64_t t_stride) {
    const int64_t n4 = nwords / 4;
    uint4* g4 = reinterpret_cast<uint4*>(grid);
    for (int64_t i = t0; i < n4; i += t_stride) g4[i] = make_uint4(0u, 0u, 0u, 0u);
    for (int64_t i = n4 * 4 + t0; i < nwords; i += t_stride) grid[i] = 0u;
}

}  // namespace vox
