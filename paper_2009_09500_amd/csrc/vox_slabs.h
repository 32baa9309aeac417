// How the small bit-volume calls deal the volume's words to their workgroups
// (k_grid_slabs, vox_grid.hip).  Host and device, so that a host check runs the
// code that the kernel runs.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace vox {

// The volume is cut into `runs` runs of `words` words (the last may be shorter).
// A workgroup's run is one of these as long as the segments are spread over
// them; where a few runs would do most of the work (a drawing in one z slice is
// one run's), the runs are cut anew by an estimate of the work: a quarter of the
// workgroups by where it is, three quarters by words as before, so that none gets
// more than about 4/3 of the words (the LDS each has).
constexpr uint32_t kSlabMaxRuns = 512;
constexpr uint32_t kSlabSamples = 256;  // segments looked at for the estimate

// Room of a workgroup's run: 4/3 of the words, and what rounding adds (a boundary
// is a multiple of 32 words; a share is up to 1/kSlabMinBase too long); whole
// 16-byte units.
constexpr uint32_t kSlabMinBase = 32;
__host__ __device__ __forceinline__ constexpr uint32_t slab_room(uint32_t words) {
    return (words + words / 3u + words / kSlabMinBase + 64u) & ~3u;
}

// Work of a segment of N steps in each of `span` runs, in voxels: a hit costs as
// much as some 13 (16 384 segments of 239 / 5 voxels in one workgroup: 1.18 / 0.092
// ms).  N is clamped so that the sums below stay under 2^32.
__host__ __device__ __forceinline__ uint32_t slab_work(uint32_t N, uint32_t span) {
#if defined(__HIP_DEVICE_COMPILE__)
    const float per = __builtin_amdgcn_rcpf((float)span);
#else
    const float per = 1.0f / (float)span;
#endif
    return (uint32_t)((float)(N < (1u << 18) ? N : 1u << 18) * per) + 13u;
}

// Whether a cut by work pays where a run has `work` of n segments: the workgroup that
// has it takes some 3 ns of each of its waves a voxel (a wave has 64 of the segments
// at a time), of which a cut leaves at best what 32 words have, and beginning again
// costs 6 us.  us a call, uncut / cut: in one slice of 256^3, 60 segments of 120
// voxels 25.1 / 8.8, 1 000 of 5 voxels 8.8 / 13.2, 2 100 of them 14.8 / 12.8; in one
// slice of 64^3 (runs of 64 words), 1 500 of 30 voxels 13.9 / 17.8.
constexpr float kSlabLeastWork = 2048.0f;  // a wave
__host__ __device__ __forceinline__ bool slab_pays(float work, uint32_t n, uint32_t words) {
    const float waves = n < 16u * 64u ? (float)((n + 63u) / 64u) : 16.0f;
    return work * (float)(words - 32u) > kSlabLeastWork * waves * (float)words;
}

// What every run weighs for its words alone, and whether the estimate (the runs'
// work `load`, its sum and maximum, from `samples` of the n segments) asks for a
// cut by work: a run with more than 16 times the mean, and enough of it.  (Uniform end
// points give 1.5 times the mean, a corner of a quarter of the sides 6; cut at 6 such
// a corner took 4 000 segments in 256^3 from 14.4 to 17.5 us, since cuts within a
// slice make every slice two workgroups'.)
__host__ __device__ __forceinline__ uint32_t slab_base(uint32_t sum, uint32_t runs) {
    return 3u * ((sum + runs - 1u) / runs);
}
__host__ __device__ __forceinline__ bool slab_uneven(uint32_t sum, uint32_t max, uint32_t runs, uint32_t n,
                                                     uint32_t samples, uint32_t words) {
    // (The last: slab_base(sum, runs) >= kSlabMinBase.)
    return ((float)max * (float)runs > 16.0f * (float)sum) & slab_pays((float)max * (float)n / (float)samples, n, words) &
           (sum > runs * ((kSlabMinBase + 2u) / 3u - 1u));
}

// Whether n segments inside a volume of this longest side can have as much work in
// one run.
inline bool slab_look(int64_t n, int32_t side, int64_t words) {
    return slab_pays((float)n * (float)(side + 12), (uint32_t)n, (uint32_t)words);
}

// Weight before the r-th of `runs` boundaries, of all runs' weight `total`.
__host__ __device__ __forceinline__ uint32_t slab_target(uint32_t r, uint32_t runs, uint32_t total) {
    const uint32_t rest = total % runs;
    return r * (total / runs) + (r < rest ? r : rest);
}
// The boundary's word, in run i, which begins at weight `before` (at most
// target) and weighs `weight`.
__host__ __device__ __forceinline__ uint32_t slab_word(uint32_t target, uint32_t i, uint32_t before, uint32_t weight,
                                                       uint32_t words, uint32_t nwords) {
    const uint32_t w = i * words + (uint32_t)((uint64_t)(target - before) * words / weight);
    return (w < nwords ? w : nwords) & ~31u;
}

}  // namespace vox
