// Voxel lists: count -> scan -> offsets + tile map -> lane-per-voxel tiles.
//
// Steps of the path (arXiv 2009.09500, Section 4 lists them as host
// preprocessing followed by one kernel; here all of them run on the GPU):
//   1. count   N_i + 1 per segment ("the voxels number in the segment",
//              host step 1 of Section 4), int16 range check;
//   2. scan    exclusive prefix sum of the counts -> d_offsets (replaces the
//              paper's padding of every segment to N_max, Section 5);
//   3. tiles   each tile of kListTile consecutive output voxels learns the
//              segment holding its first voxel;
//   4. voxels  every lane computes kListPerThread consecutive voxels of the
//              flat output with the exact stepping of eq. (3), stages them
//              in LDS and the block writes the tile with 16-byte stores.
#include <type_traits>

#include "vox_device.h"
#include "vox_internal.h"

namespace vox {

// ------------------------------------------------------------------ count

// The Euclidean length N = floor(|P1 - P0|) of eq. (1) for int16 lists:
// |d|^2 < 3 * 2^32 is rounded to float and its square root, within about
// 2^-23 relative, is within one of N; the integer corrections make it exact.
// (A float root here instead of the double one of the grid kernels: the
// Euclidean list kernels measured 3-10 % faster.)
__device__ __forceinline__ uint32_t list_euclid_length(const Seg& s) {
    uint64_t ss = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int64_t d = (int64_t)s.p1[a] - (int64_t)s.p0[a];
        ss += (uint64_t)(d * d);
    }
    uint64_t r = (uint64_t)__builtin_sqrtf((float)ss);
    while (r * r > ss) --r;
    while ((r + 1) * (r + 1) <= ss) ++r;
    return (uint32_t)r;
}

// Samples of [k0, k1) (k0 < k1 <= N + 1, N >= 1) of an int16-range
// segment that start a new voxel under the Euclidean N: sample k0 from its
// remainders (one division unless k0 = 0), then one step a sample.
//
// Up to N = 32767 an axis is a 32-bit fraction f and a slope d, and moves at a
// step exactly when f + d carries (fix32_of).  A step is three adds with
// carry and one add of the (or-ed) carries.  An axis with a = N moves at every
// step, and then so does the sample.  Longer segments step their remainders.
template <bool kFromStart>
__device__ __forceinline__ uint32_t euclid_walk(const Seg& g, uint32_t N, uint32_t k0, uint32_t k1) {
    const uint32_t two_n = 2u * N;
    uint32_t ta[3], r[3];
    bool moved = k0 == 0u, tie = false;
    const float rcpd = rcp_down(two_n);
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const int32_t d = g.p1[ax] - g.p0[ax];
        const uint32_t neg = d < 0 ? 1u : 0u;
        ta[ax] = 2u * (uint32_t)(d < 0 ? -d : d);
        tie |= ta[ax] == two_n;
        if (kFromStart || k0 == 0u) {
            r[ax] = N - neg;
        } else if (N <= 32767u) {
            // 2 k0 a + N < 2^31, 2N < 2^16, quotient <= a < 2^15.
            uint32_t q;
            divmod_down(2u * k0 * (ta[ax] >> 1) + N - neg, two_n, rcpd, q, r[ax]);
        } else {
            r[ax] = (uint32_t)(((uint64_t)k0 * ta[ax] + N - neg) % two_n);
        }
        moved |= r[ax] < ta[ax];
    }
    uint32_t c = moved ? 1u : 0u;
    const uint32_t steps = k1 - k0 - 1u;
    if (tie) return c + steps;
    if (N <= 32767u) {
        const double unit = 0x1p32 / (double)two_n;
        uint32_t f[3], d[3];
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            f[ax] = fix32_of(r[ax], unit);
            d[ax] = fix32_of(ta[ax], unit);
        }
        auto step = [&] {
            const bool a = __builtin_uadd_overflow(f[0], d[0], &f[0]);
            const bool b = __builtin_uadd_overflow(f[1], d[1], &f[1]);
            const bool e = __builtin_uadd_overflow(f[2], d[2], &f[2]);
            c += (a | b | e) ? 1u : 0u;
        };
        uint32_t k = 0;
        for (; k + 8u <= steps; k += 8u) {
#pragma unroll
            for (int i = 0; i < 8; ++i) step();
        }
        for (; k < steps; ++k) step();
        return c;
    }
    uint32_t f[3];
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) f[ax] = r[ax] - two_n;
    for (uint32_t k = 0; k < steps; ++k) {
        bool mv = false;
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            const uint32_t t = f[ax] + ta[ax];
            const bool carry = t < ta[ax];
            f[ax] = carry ? t - two_n : t;
            mv |= carry;
        }
        c += mv ? 1u : 0u;
    }
    return c;
}

// Voxels of each segment under the Euclidean N of eq. (1) (consecutive
// duplicates removed): 1 + the steps k - 1 -> k, k = 1..N, that carry on
// some axis (a carry of r_a + 2a past 2N is exactly a move of that axis,
// since a <= N); 1 for a segment outside int16, which writes nothing.
// kLanes lanes share a segment, lane l walking samples [l S, (l + 1) S),
// S = ceil((N + 1) / kLanes), from one division at its first sample, and the
// lanes' counts are summed; the host takes more lanes a segment when there
// are fewer segments, so that a few long segments still spread over the
// chip.  Per axis the walk keeps f = r - 2N, whose add of 2a carries out of
// 32 bits exactly when r + 2a >= 2N.
template <bool kAligned8, int kLanes>
__global__ __launch_bounds__(kCountBlock) void k_euclid_counts(const int32_t* __restrict__ segs, int64_t n,
                                                              uint32_t* __restrict__ counts) {
    static_assert(kLanes >= 1 && kLanes <= kWave && (kWave % kLanes) == 0, "lanes a segment");
    const uint32_t sub = threadIdx.x % kLanes;
    const int64_t groups = (int64_t)gridDim.x * (kCountBlock / kLanes);
    // (Every lane of a group takes the same segments, so a group's lanes are
    // active together at the sum below.)
    for (int64_t i = ((int64_t)blockIdx.x * kCountBlock + threadIdx.x) / kLanes; i < n; i += groups) {
        const Seg g = load_seg<kAligned8>(segs, i);
        uint32_t c = 0;
        if (!in_int16(g)) {
            c = sub == 0 ? 1u : 0u;
        } else {
            const uint32_t N = list_euclid_length(g);
            const uint32_t S = (N + (uint32_t)kLanes) / (uint32_t)kLanes;
            const uint32_t k0 = sub * S;
            const uint32_t k1 = k0 + S < N + 1u ? k0 + S : N + 1u;
            if (N == 0u) {
                c = sub == 0 ? 1u : 0u;
            } else if (k0 < k1) {
                c = euclid_walk<kLanes == 1>(g, N, k0, k1);
            }
        }
#pragma unroll
        for (int o = kLanes / 2; o >= 1; o >>= 1) c += __shfl_xor(c, o, kLanes);
        if (sub == 0) counts[i] = c;
    }
}

// Flag of the header's second word: some segment is too long for the 16.16
// coordinates of the int16 lists.
constexpr int32_t kListLong = 4;
template <int kKind>
__device__ __forceinline__ bool list_long(const Seg& g) {
    return kKind == kListI16 && seg_length(g) > (int64_t)kFix16MaxN;
}

// Bitwise OR over the block.
template <int kBlock>
__device__ __forceinline__ int32_t block_or(int32_t v, int64_t* lds) {
    const int64_t bits = (__ballot(v & kStatusOutOfRange) ? kStatusOutOfRange : 0) | (__ballot(v & kListLong) ? kListLong : 0);
    if ((threadIdx.x & (kWave - 1)) == 0) lds[threadIdx.x / kWave] = bits;
    __syncthreads();
    int64_t all = 0;
#pragma unroll
    for (int i = 0; i < kBlock / kWave; ++i) all |= lds[i];
    __syncthreads();
    return (int32_t)all;
}

// The status word (range flags, capacity) and the one after it.
// host: the status and the total for the caller as well (one lane).
__device__ __forceinline__ int32_t list_status(int32_t flags, int64_t total, int64_t capacity, int32_t* status,
                                               int64_t* host) {
    int32_t st = flags & kStatusOutOfRange;
    // (capacity > 0 exactly when voxels are wanted.)
    if (capacity > 0 && total > capacity) st |= kStatusCapacity;
    if (status) {
        status[0] = st;
        status[1] = flags & kListLong;
        if (host) {
            __hip_atomic_store(&host[0], (int64_t)st, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            __hip_atomic_store(&host[1], total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
    return st;
}

// Voxel counts per segment (N + 1, or with the Euclidean N of eq. (1) the
// samples that start a new voxel) and their block sums; out-of-range flags
// (int16 lists: a coordinate outside int16; int32 lists: an axis spanning
// 2^30 or more), and whether a segment is longer than kFix16MaxN.
// (64 VGPRs at most, so that two blocks of 1024 run on a CU where there are more
// blocks than CUs, above a million segments.)
template <bool kAligned8, int kKind, int kBlock>
__global__ __launch_bounds__(kBlock, kBlock == 1024 ? 8 : 1) void k_list_count(const int32_t* __restrict__ segs,
                                                       int64_t n, uint32_t* __restrict__ counts,
                                                       int64_t* __restrict__ block_sums,
                                                       int32_t* __restrict__ block_flags, int walk) {
    __shared__ int64_t red[kBlock / kWave];
    const int64_t base = (int64_t)blockIdx.x * (kBlock * kCountPerThread);
    int64_t sum = 0;
    int32_t flag = 0;
#pragma unroll
    for (int s = 0; s < kCountPerThread; ++s) {
        int64_t i = base + (int64_t)s * kBlock + threadIdx.x;
        if (i < n) {
            Seg g = load_seg<kAligned8>(segs, i);
            const bool inr = kKind == kListI32 ? span_below_2p30(g) : in_int16(g);
            int64_t c;
            if constexpr (kKind == kListEuclid) {
                // A thread walks its segment (walk), else from k_euclid_counts.
                if (walk) {
                    const uint32_t N = inr ? list_euclid_length(g) : 0u;
                    c = !inr || N == 0u ? 1 : (int64_t)euclid_walk<true>(g, N, 0u, N + 1u);
                } else {
                    c = counts[i];
                }
            } else {
                c = seg_length(g) + 1;
            }
            flag |= (inr ? 0 : kStatusOutOfRange) | (list_long<kKind>(g) ? kListLong : 0);
            // Counts above 2^32 - 1 only arise from out-of-range input.
            counts[i] = c > 0xFFFFFFFFll ? 0xFFFFFFFFu : (uint32_t)c;
            sum += c > 0xFFFFFFFFll ? 0xFFFFFFFFll : c;
        }
    }
    sum = block_sum<kBlock>(sum, red);
    const int32_t f = block_or<kBlock>(flag, red);
    if (threadIdx.x == 0) {
        block_sums[blockIdx.x] = sum;
        block_flags[blockIdx.x] = f;
    }
}

// ------------------------------------------------------- scan of partials

constexpr int kScanBlock = 1024;

// One block: exclusive scan of the per-block sums in place, the total into
// offsets[n] and *total, and the status word (out-of-range flags of the
// count blocks, capacity).
__global__ __launch_bounds__(kScanBlock) void k_list_scan(int64_t* __restrict__ block_sums,
                                                          const int32_t* __restrict__ block_flags,
                                                          int64_t nb, int64_t* __restrict__ offsets,
                                                          int64_t n, int64_t* __restrict__ total,
                                                          int32_t* __restrict__ status,
                                                          int64_t capacity, int64_t* host) {
    __shared__ int64_t lds[kScanBlock / kWave];
    int64_t carry = 0;
    int32_t flags = 0;
    for (int64_t c0 = 0; c0 < nb; c0 += kScanBlock) {
        int64_t i = c0 + threadIdx.x;
        int64_t v = i < nb ? block_sums[i] : 0;
        flags |= i < nb ? block_flags[i] : 0;
        int64_t tot;
        int64_t ex = block_exclusive_sum<kScanBlock>(v, lds, tot);
        if (i < nb) block_sums[i] = carry + ex;
        carry += tot;
    }
    const int32_t f = block_or<kScanBlock>(flags, lds);
    if (threadIdx.x == 0) {
        offsets[n] = carry;
        *total = carry;
        list_status(f, carry, capacity, status, host);
    }
}

// --------------------------------------------------- offsets and tile map

// Threads of a block of the count and offsets kernels, four segments each: as few
// as leave at most kFusedScanMaxBlocks blocks (300 000 segments of 4 voxels 18.7 us
// a call in blocks of 512, 21.3 of 1024).
constexpr int kMidBlock = 512, kLargeBlock = 1024;
constexpr int64_t kSmallBlockSegs = 262144, kMidBlockSegs = 524288;
static int count_block(int64_t n) { return n <= kSmallBlockSegs ? kCountBlock : n <= kMidBlockSegs ? kMidBlock : kLargeBlock; }

// Count blocks up to this many: the offsets kernel sums the count blocks'
// partials itself (every block reads all of them, 12 bytes each) and the
// scan kernel is not launched.  Measured per call: 100 000 segments 0.0255
// -> 0.0225 ms, 5 000 segments 0.016 -> 0.0135 ms (blocks of 256 threads);
// 1 M segments of 65 voxels 0.0787 -> 0.0779 (of 1024).
constexpr int64_t kFusedScanMaxBlocks = 256;

// Same segment blocks as the count kernel, kCountPerThread consecutive ones a
// thread, scanned by the block; every segment then records
// itself as the first segment of each output tile whose first voxel it
// holds.  kFused: the block's prefix, the total and the status come from the
// count blocks' raw sums and flags (what k_list_scan would write; block 0
// writes offsets[n], the total and the status word), else from k_list_scan.
template <bool kFused, int kBlock>
__global__ __launch_bounds__(kBlock) void k_list_offsets(
    int64_t n, const uint32_t* __restrict__ counts, const int64_t* __restrict__ block_prefix,
    const int32_t* __restrict__ block_flags, int64_t nb, int64_t capacity,
    int64_t* __restrict__ offsets, int32_t* __restrict__ tile_seg, int64_t tile_limit,
    int64_t* __restrict__ total, int32_t* __restrict__ status, int64_t* host) {
    __shared__ int64_t lds[kBlock / kWave];
    static_assert(kCountPerThread == 4, "one 16-byte load of counts a thread");
    const int64_t i0 = ((int64_t)blockIdx.x * kBlock + threadIdx.x) * kCountPerThread;
    // (The counts are 256-byte aligned.)
    uint4 c4 = make_uint4(0u, 0u, 0u, 0u);
    if (i0 + 3 < n) {
        c4 = *reinterpret_cast<const uint4*>(counts + i0);
    } else if (i0 < n) {
        c4.x = counts[i0];
        if (i0 + 1 < n) c4.y = counts[i0 + 1];
        if (i0 + 2 < n) c4.z = counts[i0 + 2];
    }
    const uint32_t c[kCountPerThread] = {c4.x, c4.y, c4.z, c4.w};
    int64_t carry, tot;
    bool tiles;  // only needed when voxels will be written
    if constexpr (kFused) {
        int64_t pre = 0, all = 0;
        int32_t fl = 0;
        for (int64_t b = threadIdx.x; b < nb; b += kBlock) {
            const int64_t v = block_prefix[b];
            all += v;
            pre += b < (int64_t)blockIdx.x ? v : 0;
            fl |= block_flags[b];
        }
        carry = block_sum<kBlock>(pre, lds);
        tot = block_sum<kBlock>(all, lds);
        fl = block_or<kBlock>(fl, lds);
        const bool writer = blockIdx.x == 0 && threadIdx.x == 0;
        const int32_t st = list_status(fl, tot, capacity, writer ? status : nullptr, host);
        if (writer) {
            offsets[n] = tot;
            *total = tot;
        }
        tiles = tile_limit > 0 && st == 0;
    } else {
        carry = block_prefix[blockIdx.x];
        tiles = tile_limit > 0 && *status == 0;
        tot = *total;
    }
    const int64_t ntiles = tot < tile_limit * kListTile ? (tot + kListTile - 1) / kListTile : tile_limit;
    int64_t sub;
    int64_t off = carry + block_exclusive_sum<kBlock>((int64_t)c[0] + c[1] + c[2] + c[3], lds, sub);
#pragma unroll
    for (int s = 0; s < kCountPerThread; ++s) {
        if (i0 + s < n) {
            offsets[i0 + s] = off;
            if (tiles) {
                int64_t t0 = (off + kListTile - 1) / kListTile;
                int64_t t1 = (off + c[s] - 1) / kListTile;  // inclusive
                if (t1 >= ntiles) t1 = ntiles - 1;
                for (int64_t t = t0; t <= t1; ++t) tile_seg[t] = (int32_t)(i0 + s);
            }
        }
        off += c[s];
    }
}

// ---------------------------------------------------- one-block lists

// A block's offsets of at most kSegsPerCountBlock segments: thread t's are
// kCountPerThread t and the ones after, c their counts and off their offsets.
// Returns the status (stored by one block) and the total.
template <bool kAligned8, int kKind>
__device__ __forceinline__ int32_t one_block_offsets(const int32_t* __restrict__ segs, int64_t n,
                                                     const uint32_t* __restrict__ counts, int64_t capacity,
                                                     bool store, int64_t* __restrict__ offsets,
                                                     int64_t* __restrict__ total_p, int32_t* __restrict__ status,
                                                     int64_t* host, int64_t (&c)[kCountPerThread], int64_t (&off)[kCountPerThread],
                                                     int32_t& flags, int64_t& total) {
    __shared__ int64_t lds[kCountBlock / kWave];
    int64_t sum = 0;
    int32_t flag = 0;
#pragma unroll
    for (int s = 0; s < kCountPerThread; ++s) {
        const int64_t i = (int64_t)threadIdx.x * kCountPerThread + s;
        c[s] = 0;
        off[s] = sum;
        if (i < n) {
            Seg g = load_seg<kAligned8>(segs, i);
            const bool inr = kKind == kListI32 ? span_below_2p30(g) : in_int16(g);
            int64_t v;
            if constexpr (kKind == kListEuclid) {
                v = counts[i];  // from k_euclid_counts
            } else {
                v = seg_length(g) + 1;
            }
            flag |= (inr ? 0 : kStatusOutOfRange) | (list_long<kKind>(g) ? kListLong : 0);
            c[s] = v > 0xFFFFFFFFll ? 0xFFFFFFFFll : v;
        }
        sum += c[s];
    }
    flags = block_or<kCountBlock>(flag, lds);
    const int64_t ex = block_exclusive_sum<kCountBlock>(sum, lds, total);
    const bool writer = store && threadIdx.x == 0;
    const int32_t st = list_status(flags, total, capacity, writer ? status : nullptr, host);
#pragma unroll
    for (int s = 0; s < kCountPerThread; ++s) {
        const int64_t i = (int64_t)threadIdx.x * kCountPerThread + s;
        off[s] += ex;
        if (store && i < n) offsets[i] = off[s];
    }
    if (writer) {
        offsets[n] = total;
        *total_p = total;
    }
    return st;
}

// Lists of at most kSegsPerCountBlock segments: the count, scan and offsets
// kernels in one block (a call is then two launches with the voxel kernel).
// Writes offsets[0..n], the total and the status word (range flags, capacity).
template <bool kAligned8, int kKind>
__global__ __launch_bounds__(kCountBlock) void k_list_one_block(
    const int32_t* __restrict__ segs, int64_t n, const uint32_t* __restrict__ counts,
    int64_t* __restrict__ offsets, int64_t* __restrict__ total_p, int32_t* __restrict__ status,
    int64_t* host, int64_t capacity) {
    int64_t c[kCountPerThread], off[kCountPerThread], total;
    int32_t flags;
    one_block_offsets<kAligned8, kKind>(segs, n, counts, capacity, true, offsets, total_p, status, host, c, off, flags,
                                        total);
}

static_assert(kSmallBlockSegs <= kFusedScanMaxBlocks * kSegsPerCountBlock &&
                  kMidBlockSegs <= kFusedScanMaxBlocks * kMidBlock * kCountPerThread,
              "smaller blocks are always fused");

// ------------------------------------------------------------ voxel tiles

// One tile = kListTile consecutive output voxels [j0, j1).  Its segments
// s0..s1 are staged in LDS, at most kWinSegs at a time, each as its
// stepping state at k = 0 (SegStart) with its offset relative to j0; lane t
// computes voxels j0 + t*P .. j0 + t*P + P - 1 (P = kListPerThread),
// stepping exactly from one voxel to the next and loading the following
// segment's state when the voxel index reaches its offset.  A tile with
// more segments than a window holds (segments shorter than kListTile /
// kWinSegs voxels on average) is done in several windows, each lane
// computing the voxels of its P that fall in the window; LDS sized for the
// usual case keeps many blocks on a CU.
//
// The stepping of eq. (3) per axis, for direction sign m (0 or all ones)
// and r = (2 k a + N - neg) mod 2N: the coordinate is kept as c' = c ^ m,
// which grows by one on every carry whichever the sign (for m = all ones,
// c' = -c - 1), and the remainder as f = r - 2N (mod 2^32), so that
// f + 2a carries out of 32 bits exactly when r + 2a >= 2N: one add with
// carry, one add of the carry to c', one conditional subtract of 2N.
struct SegStart {
    uint32_t c[3];     // p0 ^ m per axis
    uint32_t f[3];     // r(0) - 2N = N - neg - 2N (0 for a point)
    uint32_t ta[3];    // 2 |d_a|
    uint32_t two_n;    // 2N
    uint32_t neg;      // sign bits of d, axis a at bit a
    uint32_t pad;
};
constexpr int kWinSegs = 256;

// How a tile finds its segments.
enum ListTiles {
    kTileMap,     // in the tile map (k_list_offsets)
    kTileSearch,  // by a search of the offsets, 64 of them at a time: two rounds
                  // up to 4096 segments; the map costs a launch (1024 int32
                  // segments of 20 000 voxels: 0.0541 ms a call with it,
                  // 0.0514 without)
    kTileAll,     // every block computes all offsets (one_block_offsets) and
                  // block 0 stores them: the call is one launch
};

// The segments of voxels j and k >= j: the largest i with offsets[i] <= j, and
// k's.  All lanes of a wave take part.
__device__ __forceinline__ void find_segments(const int64_t* __restrict__ offsets, int64_t n, int64_t j, int64_t k,
                                              int32_t& sj, int32_t& sk) {
    int64_t at = 0, bt = 0, len = n;
    while (len > 1) {
        const int64_t step = (len + kWave - 1) / kWave;
        const int64_t a = at + step * (int64_t)__lane_id(), b = bt + step * (int64_t)__lane_id();
        const int64_t va = offsets[a < n ? a : n], vb = offsets[b < n ? b : n];
        // (Sample 0 is at or below; the others in order, offsets[n] above.)
        at += step * (__popcll(__builtin_amdgcn_ballot_w64(va <= j)) - 1);
        bt += step * (__popcll(__builtin_amdgcn_ballot_w64(vb <= k)) - 1);
        len = step;
    }
    sj = (int32_t)at;
    sk = (int32_t)bt;
}

// The high halves of two words, in one.
__device__ __forceinline__ uint32_t high_halves(int32_t lo, int32_t hi) {
    return __builtin_amdgcn_perm((uint32_t)hi, (uint32_t)lo, 0x07060302u);
}

// The staged state in 16.16 fixed point (int16 lists with no segment longer
// than kFix16MaxN, vox_device.h): a voxel is three adds, and its coordinates
// are the high halves, packed two a word by one byte permute each; moving to
// any voxel of the segment is a 64-bit multiply-add per axis.  (1 M segments of
// 65 voxels: 0.081 ms for the kernel, against 0.097 stepping remainders.)
struct SegFix {
    int32_t point[3];  // p0 + 1/2
    int32_t slope[3];  // d / N in 2^-30
    int32_t pad[2];
};

// What a call of one launch stores besides its voxels.
struct ListHeader {
    int64_t* offsets;
    int64_t* total;
    int32_t* status;
    int64_t* host;
    int64_t capacity;
};

// T = int16_t: coordinates in int16 (differences below 2^16); T = int32_t:
// every axis difference below 2^30 (checked by the count kernel).  The int16
// kernel is held to 64 VGPRs (eight waves a SIMD, which its 13 KiB of LDS
// allows); the int32 kernel's 25 KiB of LDS allows six blocks a CU anyway.
template <bool kAligned8, typename T, ListTiles kTiles>
__global__ __launch_bounds__(kListBlock) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 2 ? 8 : 1)))
void k_list_voxels(
    const int32_t* __restrict__ segs, int64_t n, const int64_t* __restrict__ offsets,
    const int32_t* __restrict__ tile_seg, T* __restrict__ voxels,
    const int64_t* __restrict__ total_p, const int32_t* __restrict__ status, ListHeader header) {
    constexpr int kSegWords = (int)(kWinSegs * sizeof(SegStart) / 4);
    constexpr int kVoxBytes = 3 * (int)sizeof(T);
    constexpr int kLaneWords = kListPerThread * kVoxBytes / 4;  // a lane's staged voxels
    constexpr int kStageWords = (int)kListTile * kVoxBytes / 4;
    // The staged segments and the output stage share LDS (the segments are
    // dead once every lane has its voxels): 13 KiB a block for int16 lists,
    // 25 KiB for int32 lists.
    __shared__ __align__(16) uint32_t lds_raw[kSegWords > kStageWords ? kSegWords : kStageWords];
    __shared__ int32_t srel[kWinSegs + 1];
    __shared__ int32_t srel_all[kTiles == kTileAll ? kSegsPerCountBlock + 1 : 1];
    SegStart* sseg = reinterpret_cast<SegStart*>(lds_raw);
    SegFix* sfix = reinterpret_cast<SegFix*>(lds_raw);
    uint32_t* stage = lds_raw;
    static_assert(sizeof(SegStart) % 16 == 0 && sizeof(SegFix) % 16 == 0 && (kListPerThread * kVoxBytes) % 4 == 0, "packing");

    const int64_t tile = blockIdx.x;
    const int64_t j0 = tile * kListTile;
    // An offset relative to j0 (a tile's own segments start within
    // [-(2^30 - 1), kListTile]).
    auto relative = [&](int64_t o) {
        const int64_t rel = o - j0;
        return (int32_t)(rel < -(1ll << 30) ? -(1ll << 30) : (rel > (1ll << 30) ? (1ll << 30) : rel));
    };
    int64_t total, j1;
    int32_t s0, s1, long_segs;
    if constexpr (kTiles == kTileAll) {
        __shared__ int32_t ends[2];
        int64_t c[kCountPerThread], off[kCountPerThread];
        int32_t flags;
        const int32_t st = one_block_offsets<kAligned8, sizeof(T) == 2 ? kListI16 : kListI32>(
            segs, n, nullptr, header.capacity, blockIdx.x == 0, header.offsets, header.total, header.status, header.host, c, off,
            flags, total);
        if (st != 0 || j0 >= total) return;
        j1 = j0 + kListTile < total ? j0 + kListTile : total;
#pragma unroll
        for (int i = 0; i < kCountPerThread; ++i) {
            const int32_t si = threadIdx.x * kCountPerThread + i;
            if (si < n) {
                srel_all[si] = relative(off[i]);
                if (off[i] <= j0 && j0 < off[i] + c[i]) ends[0] = si;
                if (off[i] < j1 && j1 <= off[i] + c[i]) ends[1] = si;
            }
        }
        if (threadIdx.x == 0) srel_all[n] = relative(total);
        __syncthreads();
        s0 = __builtin_amdgcn_readfirstlane(ends[0]);
        s1 = __builtin_amdgcn_readfirstlane(ends[1]);
        long_segs = flags & kListLong;
    } else {
        // The header and the tile's entries, loaded together (the map has an
        // entry more than the launch has tiles): one round trip before the
        // segments'.
        total = *total_p;
        const int32_t st0 = status[0];
        long_segs = status[1];
        if constexpr (kTiles == kTileMap) {
            s0 = tile_seg[tile];
            s1 = tile_seg[tile + 1];
            asm volatile("" ::"s"(total), "s"(long_segs), "s"(s0), "s"(s1));  // (all loaded before the first wait)
            if (st0 != 0 || j0 >= total) return;
            j1 = j0 + kListTile < total ? j0 + kListTile : total;
            const int64_t ntiles = (total + kListTile - 1) / kListTile;
            if (tile + 1 >= ntiles) s1 = (int32_t)(n - 1);
        } else {
            if (st0 != 0 || j0 >= total) return;
            j1 = j0 + kListTile < total ? j0 + kListTile : total;
            find_segments(offsets, n, j0, j1 - 1, s0, s1);
        }
    }
    const int nseg = s1 - s0 + 1;  // <= kListTile + 1

    const int first = threadIdx.x * kListPerThread;  // tile-relative voxel
    const int count = (int)(j1 - j0);
    T out[kListPerThread * 3];
    uint32_t packed[kListPerThread * 3 / 2];
    // Window w: the tile's segments [w, w + m); srel[i] is the offset of
    // segment w + i relative to j0 (srel[m]: of the segment after the window,
    // or the total), so the window's voxels are [srel[0], srel[m]).  Almost
    // every tile is one window (kOne: every voxel of the lane's P lies in it).
    auto stage_offsets = [&](int w, int m) {
        for (int i = threadIdx.x; i <= m; i += kListBlock) {
            if constexpr (kTiles == kTileAll) {
                srel[i] = srel_all[s0 + w + i];
            } else {
                const int64_t si = (int64_t)s0 + w + i;
                srel[i] = relative(si <= n ? offsets[si] : total);
            }
        }
    };
    // This lane's voxels [lo, hi) inside the window and the staged segment of
    // voxel lo (the largest s with srel[s] <= lo); false without voxels.
    // kOne: the tile is one window; kFull: and has kListTile voxels.
    auto lane_span = [&](int m, auto one, auto full, int& lo, int& hi, int& s) {
        lo = first;
        hi = decltype(full)::value || first + kListPerThread < count ? first + kListPerThread : count;
        if constexpr (!decltype(one)::value) {
            const int wlo = srel[0], whi = srel[m];
            lo = first > wlo ? first : wlo;
            hi = hi < whi ? hi : whi;
        }
        if (lo >= hi) return false;
        int a_ = 0, b_ = m - 1;
        while (a_ < b_) {
            const int mid = (a_ + b_ + 1) >> 1;
            if (srel[mid] <= lo) a_ = mid; else b_ = mid - 1;
        }
        s = a_;
        return true;
    };
    auto run_fixed = [&](int m, auto full) {
        const int w = 0;  // (one window: longer tiles step as below)
        for (int i = threadIdx.x; i < m; i += kListBlock) {
            const Seg g = load_seg<kAligned8>(segs, (int64_t)s0 + w + i);
            const uint32_t N = (uint32_t)seg_length(g);
            const double rcp_n = N ? 1.0 / (double)N : 0.0;
            SegFix f;
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                f.point[ax] = fix16_point(g.p0[ax]);
                f.slope[ax] = fix30_slope(g.p1[ax] - g.p0[ax], rcp_n);
            }
            f.pad[0] = f.pad[1] = 0;
            sfix[i] = f;
        }
        stage_offsets(w, m);
        __syncthreads();
        int lo, hi, s;
        if (!lane_span(m, std::integral_constant<bool, true>{}, full, lo, hi, s)) return;
        int next = srel[s + 1];
        SegFix f = sfix[s];
        int32_t v[3], d[3];
        const uint32_t k = (uint32_t)(lo - srel[s]);
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            v[ax] = fix16_at(f.point[ax], f.slope[ax], k);
            d[ax] = fix16_step(f.slope[ax]);
        }
        int32_t z_even = 0;
#pragma unroll
        for (int i = 0; i < kListPerThread; ++i) {
            const int j = first + i;
            // (Never at the first voxel, whose segment the search found; the
            // following segment is staged, as j < hi <= srel[m].)
            if (i > 0 && j >= next && j < hi) {
                ++s;
                next = srel[s + 1];
                f = sfix[s];
#pragma unroll
                for (int ax = 0; ax < 3; ++ax) {
                    v[ax] = f.point[ax];
                    d[ax] = fix16_step(f.slope[ax]);
                }
            }
            // Three words per two voxels: xy, zx, yz.
            if (i % 2 == 0) {
                packed[i / 2 * 3] = high_halves(v[0], v[1]);
                z_even = v[2];
            } else {
                packed[i / 2 * 3 + 1] = high_halves(z_even, v[0]);
                packed[i / 2 * 3 + 2] = high_halves(v[1], v[2]);
            }
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) v[ax] += d[ax];
        }
    };
    auto run_window = [&](int w, int m, auto one, auto full) {
        constexpr bool kOne = decltype(one)::value;
        constexpr bool kFull = decltype(full)::value;  // a tile of kListTile voxels, one window
        for (int i = threadIdx.x; i < m; i += kListBlock) {
            const Seg g = load_seg<kAligned8>(segs, (int64_t)s0 + w + i);
            SegStart st;
            uint32_t N = 0, neg[3];
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                // (int32 end points: the difference is formed without
                // overflow and is below 2^30 in magnitude.)
                const uint32_t d = (uint32_t)g.p1[ax] - (uint32_t)g.p0[ax];
                neg[ax] = (int32_t)d < 0 ? 1u : 0u;
                const uint32_t a = (int32_t)d < 0 ? 0u - d : d;
                st.ta[ax] = 2u * a;
                N = a > N ? a : N;
            }
            st.two_n = 2u * N;
            st.neg = neg[0] | (neg[1] << 1) | (neg[2] << 2);
            st.pad = 0;
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                st.c[ax] = (uint32_t)g.p0[ax] ^ (0u - neg[ax]);
                st.f[ax] = N ? (N - neg[ax]) - 2u * N : 0u;
            }
            sseg[i] = st;
        }
        stage_offsets(w, m);
        __syncthreads();

        // This lane's voxels inside the window: [lo, hi).
        int lo, hi, s;
        if (!lane_span(m, one, full, lo, hi, s)) return;
        int next = srel[s + 1];
        SegStart st = sseg[s];
        uint32_t mk[3];
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) mk[ax] = 0u - ((st.neg >> ax) & 1u);
        const uint32_t k = (uint32_t)(lo - srel[s]);
        if (k != 0u) {
            // Voxel k of the segment (k <= N, so N >= 1): c' = c'(0) + q.
            uint32_t a[3], neg[3];
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                a[ax] = st.ta[ax] >> 1;
                neg[ax] = (st.neg >> ax) & 1u;
            }
            AxisStep as[3];
            axis_init3(a, neg, st.two_n >> 1, k, as);
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                st.c[ax] += as[ax].q;
                st.f[ax] = as[ax].r - st.two_n;
            }
        }
#pragma unroll
        for (int v = 0; v < kListPerThread; ++v) {
            const int j = first + v;
            if (j >= hi || (!kOne && j < lo)) continue;
            // (Never at j = lo: the search found the segment holding voxel
            // lo, and every segment has at least one voxel.)
            if (j > lo && j >= next) {
                // First voxel of the following segment (inside the window, as
                // j < hi <= srel[m]): its state at k = 0.
                ++s;
                next = srel[s + 1];
                st = sseg[s];
#pragma unroll
                for (int ax = 0; ax < 3; ++ax) mk[ax] = 0u - ((st.neg >> ax) & 1u);
            }
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                out[v * 3 + ax] = (T)(int32_t)(st.c[ax] ^ mk[ax]);
                const uint32_t t = st.f[ax] + st.ta[ax];
                const bool carry = t < st.ta[ax];
                st.f[ax] = carry ? t - st.two_n : t;
                st.c[ax] += carry ? 1u : 0u;
            }
        }
    };
    const bool fixed = sizeof(T) == 2 && long_segs == 0 && nseg <= kWinSegs;
    if (fixed && count == (int)kListTile) {
        run_fixed(nseg, std::integral_constant<bool, true>{});
    } else if (fixed) {
        run_fixed(nseg, std::integral_constant<bool, false>{});
    } else if (nseg <= kWinSegs && count == (int)kListTile) {
        run_window(0, nseg, std::integral_constant<bool, true>{}, std::integral_constant<bool, true>{});
    } else if (nseg <= kWinSegs) {
        run_window(0, nseg, std::integral_constant<bool, true>{}, std::integral_constant<bool, false>{});
    } else {
        for (int w = 0; w < nseg; w += kWinSegs) {
            if (w > 0) __syncthreads();  // the previous window is read
            run_window(w, nseg - w < kWinSegs ? nseg - w : kWinSegs, std::integral_constant<bool, false>{},
                       std::integral_constant<bool, false>{});
        }
    }
    __syncthreads();  // the staged segments are dead from here
    if (first < count) {
        // Stage: lane t owns its 3*P coordinates, kLaneWords words at word
        // kLaneWords*t.
        uint32_t* dst = stage + kLaneWords * threadIdx.x;
        if constexpr (sizeof(T) == 2) {
            if (!fixed) {
#pragma unroll
                for (int w = 0; w < kLaneWords; ++w)
                    packed[w] = (uint32_t)(uint16_t)out[2 * w] | ((uint32_t)(uint16_t)out[2 * w + 1] << 16);
            }
#pragma unroll
            for (int w = 0; w < kLaneWords; ++w) dst[w] = packed[w];
        } else {
#pragma unroll
            for (int w = 0; w < kLaneWords; ++w) dst[w] = (uint32_t)out[w];
        }
    }
    __syncthreads();

    // Write the tile: bytes [B*j0, B*j1), B = 3*sizeof(T).  j0 is a multiple
    // of kListTile, so the start is 16-byte aligned whenever `voxels` is.
    // The stores bypass the caches (whole 128-byte lines, read by nobody here,
    // and a list larger than the caches would only push its segments and
    // offsets out of them): a whole call of 68 M voxels takes 78 us against 107,
    // one of 20 M in int32 54 against 56.
    const int64_t bytes = kVoxBytes * (j1 - j0);
    uint8_t* gbase = reinterpret_cast<uint8_t*>(voxels) + kVoxBytes * j0;
    const int64_t n16 = bytes / 16;
    typedef uint32_t Words4 __attribute__((ext_vector_type(4)));
    const Words4* src = reinterpret_cast<const Words4*>(stage);
    Words4* gdst = reinterpret_cast<Words4*>(gbase);
    for (int64_t c = threadIdx.x; c < n16; c += kListBlock) __builtin_nontemporal_store(src[c], gdst + c);
    // Tail (only in the last tile): 2-byte pieces.
    const int64_t tail0 = n16 * 16;
    const uint16_t* src16 = reinterpret_cast<const uint16_t*>(stage);
    uint16_t* dst16 = reinterpret_cast<uint16_t*>(gbase);
    for (int64_t c = tail0 / 2 + threadIdx.x; c < bytes / 2; c += kListBlock) dst16[c] = src16[c];
}

// The samples k, k + L, k + 2L, ... of one segment under the Euclidean N as
// taken by one of its L = kLanes lanes, stepped as the tile kernel steps (per axis:
// c' = coordinate ^ sign mask grows by dq + carry, f = r - 2N carries out of
// 32 bits exactly when r + dr >= 2N).  A sample k >= 1 starts a new voxel
// when some axis moved from k - 1 to k, that is when r_a(k) < 2a_a for some
// a, i.e. f_a < 2a_a - 2N as signed values (|2N| < 2^31).
struct ListSamples {
    uint32_t c[3], f[3], h[3], dq[3], dr[3], mk[3];
    uint32_t N, two_n;

    // Sample k of segment g (length n); returns whether it starts a voxel.
    __device__ __forceinline__ bool start(const Seg& g, uint32_t n, uint32_t k) {
        N = n;
        two_n = 2u * n;
        uint32_t two_a[3], num0[3];
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            const int32_t d = g.p1[ax] - g.p0[ax];
            mk[ax] = d < 0 ? ~0u : 0u;
            two_a[ax] = 2u * (uint32_t)(d < 0 ? -d : d);
            num0[ax] = n - (d < 0 ? 1u : 0u);
            h[ax] = two_a[ax] - two_n;
        }
        uint32_t q[3], r[3];
        if (n == 0) {
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) q[ax] = r[ax] = dq[ax] = dr[ax] = 0;
        } else if (n <= 32767u) {
            const float rcpd = rcp_down(two_n);
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                divmod_down(__umul24(k, two_a[ax]) + num0[ax], two_n, rcpd, q[ax], r[ax]);
                divmod_down(kWave * two_a[ax], two_n, rcpd, dq[ax], dr[ax]);
            }
        } else {
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                const uint64_t num = (uint64_t)k * two_a[ax] + num0[ax];
                q[ax] = (uint32_t)(num / two_n);
                r[ax] = (uint32_t)(num - (uint64_t)q[ax] * two_n);
                const uint32_t s = kWave * two_a[ax];
                dq[ax] = s / two_n;
                dr[ax] = s - dq[ax] * two_n;
            }
        }
        bool moved = k == 0;
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            c[ax] = ((uint32_t)g.p0[ax] ^ mk[ax]) + q[ax];
            f[ax] = r[ax] - two_n;
            moved |= (int32_t)f[ax] < (int32_t)h[ax];
        }
        return moved;
    }

    // Moves on by kLanes samples; returns whether the sample starts a voxel.
    __device__ __forceinline__ bool next() {
        bool moved = false;
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            const uint32_t t = f[ax] + dr[ax];
            const bool carry = t < dr[ax];
            f[ax] = carry ? t - two_n : t;
            c[ax] += dq[ax] + (carry ? 1u : 0u);
            moved |= (int32_t)f[ax] < (int32_t)h[ax];
        }
        return moved;
    }

    __device__ __forceinline__ int32_t coord(int ax) const { return (int32_t)(c[ax] ^ mk[ax]); }
};

// The Euclidean voxels of a segment of any int16 length, by a wave: the lanes
// take its samples 64 at a time, each stepping its own samples and deciding
// alone whether its sample starts a new voxel (ListSamples); a ballot of those
// decisions places the kept voxels, and consecutive lanes write consecutive
// voxels.  Returns their number.
__device__ __forceinline__ uint32_t euclid_voxels_any(const Seg& g, int16_t* out) {
    const uint32_t lane = __lane_id();
    ListSamples s;
    bool moved = s.start(g, list_euclid_length(g), lane);
    uint32_t rows = 0;
    for (uint32_t c0 = 0; c0 <= s.N; c0 += kWave) {
        if (c0 != 0) moved = s.next();
        const bool keep = moved && c0 + lane <= s.N;
        const uint64_t m = __builtin_amdgcn_ballot_w64(keep);
        if (keep) {
            const uint32_t before = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                              __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            int16_t* o = out + 3 * (uint64_t)(rows + before);
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) o[ax] = (int16_t)s.coord(ax);
        }
        rows += (uint32_t)__popcll(m);
    }
    return rows;
}

// Lists with the Euclidean N of eq. (1).  A wave takes up to 64 consecutive
// segments: a lane each for what depends on the segment alone (LDS), then kL
// lanes each for the samples, a run of up to kEuclidRun consecutive ones a
// lane; a longer segment takes all lanes, window by window, and kL is what gives
// the wave the fewest passes (2 M segments of 1 to 45 samples: 0.109 ms, 0.152
// where all but four of the wave's segments had to fit one run a lane).  Per axis the
// coordinate at sample k is the high word of start + k slope (64 bits), the
// fraction its low word, and a step's carry out of the fraction is a move of
// the axis, so the kept samples of a run are counted with three adds a sample,
// and after a scan of the counts over the lanes a second walk puts them in
// place: six adds, the packing of a row and two LDS writes a sample.  (Lanes
// stepping strided samples and a ballot for every 64 took 28 instructions a
// sample, and 0.196 ms for 1 M segments of 64 samples; this one 0.131 ms, and
// 0.177 against 0.323 ms for 11 M segments of 5 samples.)
//
// (Exact: fix32_slope, fix32_at.)
//
// The wave's output is contiguous: rows go through an LDS buffer, x and y apart
// from z (rows of 6 bytes would take unaligned writes, five times as slow), and
// from there to memory, two rows a lane, in whole 128-byte lines past the caches
// (0.147 ms a call of 1 M segments of 64-110 samples, against 0.157 through
// them; lines written in parts past them 0.182).  What bounds it: about 350
// instructions a group of 64 lanes, 60 % of the issue slots, and their latency.
// Runs of 7 / 9 / 11 / 15 (less LDS, more waves, against fewer set-ups a sample):
// 0.139 / 0.144 / 0.156 / 0.148 ms, but 0.161 / 0.126 / 0.125 / 0.150 for the
// kernel on 400 000 segments of 171 samples.
constexpr uint32_t kEuclidMaxN = 32767;
constexpr uint32_t kEuclidRun = 9;                        // samples of a lane at a time
constexpr uint32_t kEuclidBuffer = kWave * kEuclidRun;    // rows
constexpr uint32_t kEuclidGroup = 64;                     // rows of whole 128-byte lines of memory: 3 x 128 / 6
struct EuclidSeg {
    uint32_t c[3];      // p0 ^ m, m the sign mask of d (c' = c ^ m grows by one on every move)
    uint32_t slope[3];  // a / N
    uint32_t n_neg;     // N | sign bits of d << 24
    uint32_t start;     // 2^-32 / 2N units of the start of a negative axis: 1/2 - 1/2N
};
struct EuclidWave {
    EuclidSeg seg[kWave];
    __align__(16) uint32_t xy[kEuclidBuffer + kEuclidGroup];
    __align__(16) uint16_t z[kEuclidBuffer + kEuclidGroup];
};

template <bool kAligned8>
struct EuclidLists {
    EuclidWave& w;
    int16_t* voxels;
    int64_t base;       // the wave's first voxel
    uint32_t from = 0, to = 0;  // voxels in the buffer, relative to base

    static __device__ __forceinline__ void fence() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }

    // Place in the buffer of voxel base + v: groups of places are groups of
    // the list's rows.
    __device__ __forceinline__ uint32_t place(uint32_t v) const {
        return ((uint32_t)(base + from) % kEuclidGroup) + (v - from);
    }

    // Writes the buffer's whole groups of rows, or all rows.
    __device__ __forceinline__ void flush(bool all) {
        const uint32_t h0 = place(from), h2 = place(to), h1 = all ? h2 : h2 / kEuclidGroup * kEuclidGroup;
        if (h1 <= h0) return;
        fence();
        const uint32_t lane = __lane_id();
        int16_t* dst = voxels + 3 * (base + from - h0);
        // Four units a lane in flight.
        constexpr uint32_t kUnits = 4;
        for (uint32_t u0 = (h0 + 1u) / 2u + lane; u0 < h1 / 2u; u0 += kWave * kUnits) {
            uint2 p[kUnits];
            uint32_t q[kUnits];
#pragma unroll
            for (uint32_t i = 0; i < kUnits; ++i) {
                const uint32_t u = u0 + i * kWave < (kEuclidBuffer + kEuclidGroup) / 2u ? u0 + i * kWave : 0u;
                p[i] = reinterpret_cast<const uint2*>(w.xy)[u];
                q[i] = reinterpret_cast<const uint32_t*>(w.z)[u];
            }
#pragma unroll
            for (uint32_t i = 0; i < kUnits; ++i) {
                const uint32_t u = u0 + i * kWave;
                if (u < h1 / 2u) {
                    uint32_t* row2 = reinterpret_cast<uint32_t*>(dst) + 3u * u;
                    __builtin_nontemporal_store(p[i].x, row2);
                    __builtin_nontemporal_store((q[i] & 0xFFFFu) | (p[i].y << 16), row2 + 1);
                    __builtin_nontemporal_store((p[i].y >> 16) | (q[i] & 0xFFFF0000u), row2 + 2);
                }
            }
        }
        // A row whose pair is not here, first or last.
        const uint32_t odd = lane == 0 ? h0 : h1 - 1u;
        if ((lane == 0 && (h0 & 1u) != 0u) || (lane == 1 && (h1 & 1u) != 0u)) {
            dst[3 * odd] = (int16_t)w.xy[odd];
            dst[3 * odd + 1] = (int16_t)(w.xy[odd] >> 16);
            dst[3 * odd + 2] = (int16_t)w.z[odd];
        }
        // The rows of the group begun move to its place at the front.
        const uint32_t left = h1 + lane < h2 ? h1 + lane : h0;
        const uint32_t xy = w.xy[left];
        const uint16_t z = w.z[left];
        fence();
        if (h1 + lane < h2) {
            w.xy[lane] = xy;
            w.z[lane] = z;
        }
        fence();
        from += h1 - h0;
    }

    // Samples [win, win + kL kEuclidRun) of segments [s0, s0 + 64 / kL) of the
    // wave's (below cnt), whose rows follow the buffer's last one; returns the
    // number of rows.
    template <int kL>
    __device__ __forceinline__ uint32_t run(uint32_t s0, uint32_t cnt, uint32_t win, uint32_t at) {
        const uint32_t lane = __lane_id(), sub = lane % kL, slot = lane / kL;
        const bool valid = s0 + slot < cnt;
        const EuclidSeg e = w.seg[valid ? s0 + slot : s0];
        const uint32_t N = e.n_neg & 0xFFFFFFu;
        // This lane's samples [k0, k0 + len).
        const uint32_t left = N + 1u - win, share = left < kL * kEuclidRun ? (left + kL - 1u) / kL : kEuclidRun;
        const uint32_t k0 = win + sub * share;
        const uint32_t len = !valid || k0 > N ? 0u : (N + 1u - k0 < share ? N + 1u - k0 : share);
        uint32_t c[3], f[3], g[3], mk[3];
        bool kept = k0 == 0u;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const bool neg = ((e.n_neg >> (24 + a)) & 1u) != 0u;
            mk[a] = neg ? ~0u : 0u;
            const uint64_t t = fix32_at(k0, e.slope[a], neg, e.start);
            c[a] = e.c[a] + (uint32_t)(t >> 32);
            f[a] = g[a] = (uint32_t)t;
            kept |= f[a] < e.slope[a];  // the step to k0 carried
        }
        kept &= len != 0u;
        uint32_t rows = kept ? 1u : 0u;
        for (uint32_t j = 1; j < len; ++j) {
            const bool x = __builtin_uadd_overflow(g[0], e.slope[0], &g[0]);
            const bool y = __builtin_uadd_overflow(g[1], e.slope[1], &g[1]);
            const bool z = __builtin_uadd_overflow(g[2], e.slope[2], &g[2]);
            rows += (x | y | z) ? 1u : 0u;
        }
        const uint32_t incl = wave_inclusive_sum_dpp(rows);
        uint32_t o = at + (incl - rows);
        const uint32_t mxy = (mk[0] & 0xFFFFu) | (mk[1] << 16);
        auto put = [&] {
            w.xy[o] = __builtin_amdgcn_perm(c[1], c[0], 0x05040100u) ^ mxy;
            w.z[o] = (uint16_t)(c[2] ^ mk[2]);
            ++o;
        };
        if (kept) put();
        for (uint32_t j = 1; j < len; ++j) {
            const bool x = __builtin_uadd_overflow(f[0], e.slope[0], &f[0]);
            const bool y = __builtin_uadd_overflow(f[1], e.slope[1], &f[1]);
            const bool z = __builtin_uadd_overflow(f[2], e.slope[2], &f[2]);
            c[0] += x ? 1u : 0u;
            c[1] += y ? 1u : 0u;
            c[2] += z ? 1u : 0u;
            if (x | y | z) put();
        }
        return __builtin_amdgcn_readlane(incl, kWave - 1);
    }

    // Segment t of the wave's, of length n, with all lanes.
    __device__ __forceinline__ void one(const int32_t* __restrict__ segs, int64_t i0, uint32_t t, uint32_t n) {
        if (n > kEuclidMaxN) {
            flush(true);
            to += euclid_voxels_any(load_seg<kAligned8>(segs, i0 + t), voxels + 3 * (base + to));
            from = to;
        } else {
            for (uint32_t win = 0; win <= n; win += kWave * kEuclidRun) {
                to += run<kWave>(t, t + 1u, win, place(to));
                flush(false);
            }
        }
    }

    // The wave's cnt segments, kL lanes each; lane t holds the N of segment t.
    template <int kL>
    __device__ __forceinline__ void groups(const int32_t* __restrict__ segs, int64_t i0, uint32_t cnt, uint32_t N) {
        constexpr uint32_t kSlots = kWave / kL;
        const uint64_t longer = __builtin_amdgcn_ballot_w64((uint32_t)__lane_id() < cnt && N >= kL * kEuclidRun);
        for (uint32_t s = 0; s < cnt;) {
            const uint64_t rest = longer >> s;
            if ((rest & 1u) != 0) {
                one(segs, i0, s, __builtin_amdgcn_readlane(N, s));
                ++s;
            } else {
                // Those up to the next longer one, as many as the lanes take.
                uint32_t end = rest ? s + (uint32_t)__builtin_ctzll(rest) : cnt;
                end = end < s + kSlots ? end : s + kSlots;
                to += run<kL>(s, end, 0u, place(to));
                flush(false);
                s = end;
            }
        }
    }

    // Segments [i0, i0 + cnt), cnt <= 64.
    __device__ __forceinline__ void wave(const int32_t* __restrict__ segs, const int64_t* __restrict__ offsets,
                                         int64_t i0, uint32_t cnt) {
        const uint32_t lane = __lane_id();
        const int64_t i = i0 + (lane < cnt ? lane : cnt - 1u);
        const Seg g = load_seg<kAligned8>(segs, i);
        const int64_t o = offsets[i0];
        base = ((int64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(o >> 32)) << 32) |
               (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)o);
        from = to = 0u;
        const uint32_t N = list_euclid_length(g);
        const double rcp_n = N ? 1.0 / (double)N : 0.0;
        EuclidSeg e;
        e.n_neg = N;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int32_t d = g.p1[a] - g.p0[a];
            const uint32_t len = (uint32_t)(d < 0 ? -d : d);
            e.c[a] = (uint32_t)g.p0[a] ^ (d < 0 ? ~0u : 0u);
            e.slope[a] = fix32_slope(len, N, rcp_n);
            e.n_neg |= d < 0 ? 1u << (24 + a) : 0u;
        }
        e.start = fix32_start(rcp_n);
        w.seg[lane] = e;
        fence();
        // Lanes a segment: the fewest passes over the wave's segments, those
        // that are longer than one run a lane one by one (and half a pass
        // lost before each), the others 64 / lanes at a time.
        uint32_t lanes = kWave, best = ~0u;
#pragma unroll
        for (uint32_t l = 1; l <= (uint32_t)kWave; l *= 2u) {
            const uint32_t big = (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(lane < cnt && N >= l * kEuclidRun));
            const uint32_t cost = big * 64u + (cnt - big) * l + (big < cnt - big ? big : cnt - big) * 32u;
            // (As many lanes as spread few segments over the wave.)
            if (l * cnt > kWave / 2u && cost < best) {
                best = cost;
                lanes = l;
            }
        }
        switch (lanes) {
            case 1: groups<1>(segs, i0, cnt, N); break;
            case 2: groups<2>(segs, i0, cnt, N); break;
            case 4: groups<4>(segs, i0, cnt, N); break;
            case 8: groups<8>(segs, i0, cnt, N); break;
            case 16: groups<16>(segs, i0, cnt, N); break;
            case 32: groups<32>(segs, i0, cnt, N); break;
            default: groups<64>(segs, i0, cnt, N); break;
        }
        flush(true);
        fence();  // the segments are rewritten by the wave's next ones
    }
};

template <bool kAligned8>
__global__ __launch_bounds__(kCountBlock) void k_list_voxels_euclid(
    const int32_t* __restrict__ segs, int64_t n, const int64_t* __restrict__ offsets,
    int16_t* __restrict__ voxels, const int32_t* __restrict__ status, int32_t per_wave) {
    __shared__ EuclidWave waves[kCountBlock / kWave];
    if (status[0] != 0) return;
    const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    EuclidLists<kAligned8> lists{waves[wv], voxels, 0};
    constexpr int kWaves = kCountBlock / kWave;
    const int64_t step = (int64_t)gridDim.x * kWaves * per_wave;
    for (int64_t i0 = ((int64_t)blockIdx.x * kWaves + wv) * per_wave; i0 < n; i0 += step)
        lists.wave(segs, offsets, i0, n - i0 < per_wave ? (uint32_t)(n - i0) : (uint32_t)per_wave);
}

template <bool kAligned8>
__global__ __launch_bounds__(kCountBlock) void k_list_voxels_euclid_any(
    const int32_t* __restrict__ segs, int64_t n, const int64_t* __restrict__ offsets,
    int16_t* __restrict__ voxels, const int32_t* __restrict__ status) {
    if (status[0] != 0) return;
    constexpr int kWaves = kCountBlock / kWave;
    const int64_t step = (int64_t)gridDim.x * kWaves;
    for (int64_t i = (int64_t)blockIdx.x * kWaves + threadIdx.x / kWave; i < n; i += step)
        euclid_voxels_any(load_seg<kAligned8>(segs, i), voxels + 3 * offsets[i]);
}

// ---------------------------------------------------------------- host side

size_t list_workspace_bytes(int64_t n, int64_t capacity) {
    int64_t nb = (n + kSegsPerCountBlock - 1) / kSegsPerCountBlock;
    if (nb < 1) nb = 1;
    int64_t ntiles = (capacity + kListTile - 1) / kListTile;
    size_t b = kAlign;                                  // status, total
    b += align_up((size_t)nb * sizeof(int64_t));         // block sums
    b += align_up((size_t)nb * sizeof(int32_t));         // block flags
    b += align_up((size_t)(n > 0 ? n : 1) * sizeof(uint32_t));  // counts
    b += align_up((size_t)(ntiles + 1) * sizeof(int32_t));      // tile map
    return b;
}

ListWork list_workspace(void* d_work, int64_t n, int64_t capacity) {
    ListWork w;
    int64_t nb = (n + kSegsPerCountBlock - 1) / kSegsPerCountBlock;
    if (nb < 1) nb = 1;
    uint8_t* p = static_cast<uint8_t*>(d_work);
    w.status = reinterpret_cast<int32_t*>(p);
    w.total = reinterpret_cast<int64_t*>(p + 8);
    p += kAlign;
    w.block_sums = reinterpret_cast<int64_t*>(p);
    p += align_up((size_t)nb * sizeof(int64_t));
    w.block_flags = reinterpret_cast<int32_t*>(p);
    p += align_up((size_t)nb * sizeof(int32_t));
    w.counts = reinterpret_cast<uint32_t*>(p);
    p += align_up((size_t)(n > 0 ? n : 1) * sizeof(uint32_t));
    w.tile_seg = reinterpret_cast<int32_t*>(p);
    const int64_t per = (int64_t)count_block(n) * kCountPerThread;
    w.nb = n > 0 ? (n + per - 1) / per : 1;
    w.ntiles = (capacity + kListTile - 1) / kListTile;
    return w;
}

template <int kLanes>
static void euclid_counts(const int32_t* segs, int64_t n, bool aligned8, uint32_t* counts, hipStream_t stream) {
    int64_t blocks = (n * kLanes + kCountBlock - 1) / kCountBlock;
    if (blocks > 16384) blocks = 16384;
    if (aligned8)
        k_euclid_counts<true, kLanes><<<dim3((unsigned)blocks), kCountBlock, 0, stream>>>(segs, n, counts);
    else
        k_euclid_counts<false, kLanes><<<dim3((unsigned)blocks), kCountBlock, 0, stream>>>(segs, n, counts);
}

// Euclidean counts into w.counts (n >= 1): one lane a segment from 65 536
// segments on (a thread per segment already fills the chip), more lanes a
// segment below that, and more again while a lane would walk more than
// about 256 samples (voxels a segment taken from the caller's capacity, the
// workspace's tile count; none when only the total is asked for).
static int euclid_count_lanes(int64_t n, const ListWork& w) {
    int lanes = n >= 65536 ? 1 : (n >= 16384 ? 4 : (n >= 4096 ? 16 : 64));
    const int64_t avg = w.ntiles * kListTile / n;
    while (lanes < kWave && (int64_t)lanes * 256 < avg) lanes *= 4;
    return lanes;
}

static void launch_euclid_counts(const int32_t* segs, int64_t n, bool aligned8, const ListWork& w,
                                 hipStream_t stream) {
    const int lanes = euclid_count_lanes(n, w);
    if (lanes == 1)
        euclid_counts<1>(segs, n, aligned8, w.counts, stream);
    else if (lanes == 4)
        euclid_counts<4>(segs, n, aligned8, w.counts, stream);
    else if (lanes == 16)
        euclid_counts<16>(segs, n, aligned8, w.counts, stream);
    else
        euclid_counts<64>(segs, n, aligned8, w.counts, stream);
}

// With one lane a segment the count kernel may walk the segments itself, one launch
// fewer, but four a thread, a wave as long as its longest.  us a call, walking /
// not: 400 000 segments of 4 voxels 27 / 27, of 40 at 500 000 68 / 65, 1.3 M 131 /
// 129, 2 M 178 / 187, 4 M 334 / 355; of 64 to 110 at 1.3 M 195 / 190, 2 M 271 / 277;
// of 1 to 400 mixed at 1.3 M 377 / 326, 2 M 479 / 472; 100 000 of 1 to 960 209 / 105.
// A call that asks for the total alone says nothing of the lengths: of 4 at 65 536
// 22 / 23, 1 M 33 / 38, 2 M 45 / 53, but of 1 to 900 166 / 66 at 65 536, of 1 to 400
// 110 / 97 at 1 M and 171 / 161 at 2 M.
constexpr int64_t kWalkVoxels = 32;                     // a segment, by the capacity
constexpr int64_t kWalkManyVoxels = 64, kWalkManySegs = int64_t(1) << 21;

static bool walk_in_count(int64_t n, const ListWork& w) {
    if (n == 0 || euclid_count_lanes(n, w) != 1) return false;
    const int64_t room = w.ntiles * kListTile;
    if (room == 0) return n >= kWalkManySegs;
    return room <= kWalkVoxels * n || (n >= kWalkManySegs && room <= kWalkManyVoxels * n);
}

template <int kKind>
static void list_count(const int32_t* segs, int64_t n, bool aligned8, const ListWork& w, hipStream_t stream) {
    const int walk = kKind == kListEuclid && walk_in_count(n, w) ? 1 : 0;
    if (kKind == kListEuclid && n > 0 && !walk) launch_euclid_counts(segs, n, aligned8, w, stream);
    // n == 0: one block that writes a zero sum and no flag.
    dim3 grid(n == 0 ? 1u : (unsigned)w.nb);
    auto launch = [&](auto block) {
        constexpr int kBlock = decltype(block)::value;
        if (aligned8)
            k_list_count<true, kKind, kBlock><<<grid, kBlock, 0, stream>>>(segs, n, w.counts, w.block_sums,
                                                                           w.block_flags, walk);
        else
            k_list_count<false, kKind, kBlock><<<grid, kBlock, 0, stream>>>(segs, n, w.counts, w.block_sums,
                                                                            w.block_flags, walk);
    };
    if (count_block(n) == kLargeBlock)
        launch(std::integral_constant<int, kLargeBlock>{});
    else if (count_block(n) == kMidBlock)
        launch(std::integral_constant<int, kMidBlock>{});
    else
        launch(std::integral_constant<int, kCountBlock>{});
}

hipError_t launch_list_count(const int32_t* segs, int64_t n, bool aligned8, const ListWork& w,
                             hipStream_t stream, ListKind kind) {
    KernelTimer timer(kind == kListEuclid ? "list_count_euclid" : (kind == kListI32 ? "list_count32" : "list_count"),
                      stream);
    if (kind == kListEuclid)
        list_count<kListEuclid>(segs, n, aligned8, w, stream);
    else if (kind == kListI32)
        list_count<kListI32>(segs, n, aligned8, w, stream);
    else
        list_count<kListI16>(segs, n, aligned8, w, stream);
    return hipGetLastError();
}

template <int kKind>
static void list_one_block(const int32_t* segs, int64_t n, bool aligned8, const ListWork& w, int64_t* offsets,
                           int64_t capacity, hipStream_t stream) {
    if (kKind == kListEuclid && n > 0) launch_euclid_counts(segs, n, aligned8, w, stream);
    if (aligned8)
        k_list_one_block<true, kKind><<<1, kCountBlock, 0, stream>>>(segs, n, w.counts, offsets, w.total, w.status,
                                                                      w.host, capacity);
    else
        k_list_one_block<false, kKind><<<1, kCountBlock, 0, stream>>>(segs, n, w.counts, offsets, w.total,
                                                                       w.status, w.host, capacity);
}

// Whether the tiles of a list with room for this many search for their
// segments, or find them in the map.
static bool list_searches(int64_t n, int64_t tiles) { return n <= kSegsPerCountBlock || tiles > 4 * n; }

// Lists of one launch: up to two blocks a CU, each of which computes all
// offsets (1000 segments, 70 tiles: 0.0116 -> 0.0082 ms a call, its host time).
constexpr int64_t kOneLaunchMaxTiles = 512;

hipError_t launch_list_one_block(const int32_t* segs, int64_t n, bool aligned8, const ListWork& w,
                                 int64_t* offsets, int64_t capacity, hipStream_t stream, ListKind kind) {
    KernelTimer timer("list_one_block", stream);
    if (kind == kListEuclid)
        list_one_block<kListEuclid>(segs, n, aligned8, w, offsets, capacity, stream);
    else if (kind == kListI32)
        list_one_block<kListI32>(segs, n, aligned8, w, offsets, capacity, stream);
    else
        list_one_block<kListI16>(segs, n, aligned8, w, offsets, capacity, stream);
    return hipGetLastError();
}

hipError_t launch_list_scan(const ListWork& w, int64_t n, int64_t* offsets, int64_t capacity,
                            hipStream_t stream) {
    if (n >= 1 && w.nb <= kFusedScanMaxBlocks) return hipSuccess;  // done by the offsets kernel
    KernelTimer timer("list_scan", stream);
    k_list_scan<<<1, kScanBlock, 0, stream>>>(w.block_sums, w.block_flags, w.nb, offsets, n, w.total,
                                              w.status, capacity, w.host);
    return hipGetLastError();
}

hipError_t launch_list_offsets(int64_t n, int64_t* offsets, const ListWork& w, int64_t capacity,
                               bool want_voxels, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    const int64_t tiles = want_voxels ? (capacity + kListTile - 1) / kListTile : 0;
    // (No map for segments of more than four tiles on average, whose runs of
    // entries a thread each would write: the tiles search.)
    const int64_t mapped = list_searches(n, tiles) ? 0 : tiles;
    KernelTimer timer("list_offsets", stream);
    auto launch = [&](auto fused, auto block) {
        constexpr int kBlock = decltype(block)::value;
        k_list_offsets<decltype(fused)::value, kBlock><<<dim3((unsigned)w.nb), kBlock, 0, stream>>>(
            n, w.counts, w.block_sums, w.block_flags, w.nb, capacity, offsets, w.tile_seg, mapped, w.total, w.status,
            w.host);
    };
    if (count_block(n) == kCountBlock)
        launch(std::true_type{}, std::integral_constant<int, kCountBlock>{});
    else if (count_block(n) == kMidBlock)
        launch(std::true_type{}, std::integral_constant<int, kMidBlock>{});
    else if (w.nb <= kFusedScanMaxBlocks)
        launch(std::true_type{}, std::integral_constant<int, kLargeBlock>{});
    else
        launch(std::false_type{}, std::integral_constant<int, kLargeBlock>{});
    return hipGetLastError();
}

template <typename T, ListTiles kTiles>
static void list_voxels(const int32_t* segs, int64_t n, bool aligned8, const int64_t* offsets, const ListWork& w,
                        T* voxels, int64_t tiles, const ListHeader& header, hipStream_t stream) {
    if (aligned8)
        k_list_voxels<true, T, kTiles><<<dim3((unsigned)tiles), kListBlock, 0, stream>>>(
            segs, n, offsets, w.tile_seg, voxels, w.total, w.status, header);
    else
        k_list_voxels<false, T, kTiles><<<dim3((unsigned)tiles), kListBlock, 0, stream>>>(
            segs, n, offsets, w.tile_seg, voxels, w.total, w.status, header);
}

template <typename T>
static hipError_t launch_tiles(const int32_t* segs, int64_t n, bool aligned8, const int64_t* offsets,
                               const ListWork& w, T* voxels, int64_t tiles, hipStream_t stream) {
    if (n == 0 || tiles <= 0) return hipSuccess;
    KernelTimer timer(sizeof(T) == 2 ? "list_voxels" : "list_voxels32", stream);
    if (list_searches(n, w.ntiles))
        list_voxels<T, kTileSearch>(segs, n, aligned8, offsets, w, voxels, tiles, ListHeader{}, stream);
    else
        list_voxels<T, kTileMap>(segs, n, aligned8, offsets, w, voxels, tiles, ListHeader{}, stream);
    return hipGetLastError();
}

hipError_t launch_list_voxels(const int32_t* segs, int64_t n, bool aligned8, const int64_t* offsets,
                              const ListWork& w, int16_t* voxels, int64_t tiles, hipStream_t stream) {
    return launch_tiles(segs, n, aligned8, offsets, w, voxels, tiles, stream);
}

hipError_t launch_list_voxels32(const int32_t* segs, int64_t n, bool aligned8, const int64_t* offsets,
                                const ListWork& w, int32_t* voxels, int64_t tiles, hipStream_t stream) {
    return launch_tiles(segs, n, aligned8, offsets, w, voxels, tiles, stream);
}

bool list_one_launch(int64_t n, int64_t capacity) {
    return n >= 1 && n <= kSegsPerCountBlock && capacity <= kOneLaunchMaxTiles * kListTile;
}

hipError_t launch_list_all(const int32_t* segs, int64_t n, bool aligned8, int64_t* offsets, const ListWork& w,
                           void* voxels, int64_t capacity, hipStream_t stream, ListKind kind) {
    KernelTimer timer("list_all", stream);
    const ListHeader header{offsets, w.total, w.status, w.host, capacity};
    if (kind == kListI32)
        list_voxels<int32_t, kTileAll>(segs, n, aligned8, offsets, w, static_cast<int32_t*>(voxels), w.ntiles,
                                       header, stream);
    else
        list_voxels<int16_t, kTileAll>(segs, n, aligned8, offsets, w, static_cast<int16_t*>(voxels), w.ntiles,
                                       header, stream);
    return hipGetLastError();
}

// Segments of a wave: 64 share one preparation, but few long ones spread over
// the chip.
static void list_voxels_euclid(const int32_t* segs, int64_t n, bool aligned8, const int64_t* offsets,
                               const ListWork& w, int16_t* voxels, hipStream_t stream) {
    // (Waves in all, by the voxels a segment: short ones gain more from sharing.
    // 2048 / 4096 / 8192: 30 000 segments of 20 samples 18.2 / 19.2 / 22.6 us a
    // call, 20 000 of 50 21.3 / 20.2 / 23.2, 48 000 of 1 to 2048 115 / 88 / 84.
    // 4096 / 8192: 20 000 of 64 20.2 / 23.2, of 120 23.5 / 25.4, 65 000 of 120 38.8 /
    // 38.3, 50 000 of 300 52 / 49.)
    const int64_t avg = w.ntiles * kListTile / n;
    int64_t per = n / (avg <= 32 ? 2048 : (avg <= 128 ? 4096 : 8192));
    per = per < 1 ? 1 : (per > kWave ? kWave : per);
    const int64_t segs_per_block = per * (kCountBlock / kWave);
    int64_t blocks = (n + segs_per_block - 1) / segs_per_block;
    if (blocks > 16384) blocks = 16384;
    if (aligned8)
        k_list_voxels_euclid<true><<<dim3((unsigned)blocks), kCountBlock, 0, stream>>>(
            segs, n, offsets, voxels, w.status, (int32_t)per);
    else
        k_list_voxels_euclid<false><<<dim3((unsigned)blocks), kCountBlock, 0, stream>>>(
            segs, n, offsets, voxels, w.status, (int32_t)per);
}

// Segments of more voxels than this on average (by the caller's capacity) take
// the general form with a wave each: its stores are whole rounds of 64 samples
// and it needs no LDS, hence twice the waves.  68 M voxels in segments of 500 /
// 1000 / 2000 samples: 0.130 / 0.118 / 0.107 ms against 0.127 / 0.126 / 0.127.
// So do few segments, which do not fill the chip otherwise (3 394 of 1 to 2048
// samples 24.1 against 28.3 us a call, 10 885 of 53 18.8 / 23.2; at 20 000 of 50
// 21.6 / 20.2).
constexpr int64_t kEuclidAnyVoxels = 750;
constexpr int64_t kEuclidAnySegs = 16384;

static void list_voxels_euclid_any(const int32_t* segs, int64_t n, bool aligned8, const int64_t* offsets,
                                   const ListWork& w, int16_t* voxels, hipStream_t stream) {
    int64_t blocks = (n + kCountBlock / kWave - 1) / (kCountBlock / kWave);
    if (blocks > 16384) blocks = 16384;
    if (aligned8)
        k_list_voxels_euclid_any<true><<<dim3((unsigned)blocks), kCountBlock, 0, stream>>>(segs, n, offsets,
                                                                                           voxels, w.status);
    else
        k_list_voxels_euclid_any<false><<<dim3((unsigned)blocks), kCountBlock, 0, stream>>>(segs, n, offsets,
                                                                                            voxels, w.status);
}

hipError_t launch_list_voxels_euclid(const int32_t* segs, int64_t n, bool aligned8, const int64_t* offsets,
                                     const ListWork& w, int16_t* voxels, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    KernelTimer timer("list_voxels_euclid", stream);
    if (n < kEuclidAnySegs || w.ntiles * kListTile / n > kEuclidAnyVoxels)
        list_voxels_euclid_any(segs, n, aligned8, offsets, w, voxels, stream);
    else
        list_voxels_euclid(segs, n, aligned8, offsets, w, voxels, stream);
    return hipGetLastError();
}

}  // namespace vox
