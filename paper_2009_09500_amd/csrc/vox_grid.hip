// Bit-volume output of calls the brick path does not take.  Small ones: every
// workgroup owns a run of the volume's words in LDS and takes from all
// segments the voxels that fall there (k_grid_slabs).  The others, direct
// form: every voxel is ORed into its grid word with a device-scope atomic.
// Both are correct for any volume shape.
#include "vox.h"
#include "vox_device.h"
#include "vox_direct.h"
#include "vox_exact.h"
#include "vox_internal.h"
#include "vox_slabs.h"

namespace vox {

constexpr int kGridBlock = 256;

__global__ void k_grid_init(int32_t* status) {
    if (threadIdx.x == 0) *status = 0;
}

// Zeroes the volume and the status word (a cleared direct call is then two
// launches).
__global__ __launch_bounds__(kGridBlock) void k_grid_clear(uint32_t* __restrict__ grid, int64_t nwords,
                                                           int32_t* __restrict__ status) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *status = 0;
    clear_words(grid, nwords, (int64_t)blockIdx.x * kGridBlock + threadIdx.x, (int64_t)gridDim.x * kGridBlock);
}

// All segments of one volume (direct_segments, vox_direct.h).
template <bool kAligned8, bool kEuclid, bool kRuns>
__global__ __launch_bounds__(kGridBlock) void k_grid_direct(const int32_t* __restrict__ segs, int64_t n,
                                                            int32_t dx, int32_t dy, int32_t dz,
                                                            uint32_t* __restrict__ grid,
                                                            int32_t* __restrict__ counts,
                                                            int32_t* __restrict__ status) {
    direct_segments<kAligned8, kEuclid, kRuns>(segs, n, dx, dy, dz, grid, counts, status,
                                               (int64_t)blockIdx.x * (kGridBlock / kWave) + threadIdx.x / kWave,
                                               (int64_t)gridDim.x * (kGridBlock / kWave));
}

// ------------------------------------------------------------------- slabs

// Samples of a segment that a lane takes at a time.
constexpr uint32_t kSlabChunk = 8;
constexpr int kSlabBlock = 1024;

// A wave's segments that may hold voxels of its run (a queue of fewer than 192),
// and the end points and windows of the 64 it works on.
struct SlabHits {
    uint32_t queue[3 * kWave];
    int32_t seg[6][kWave];
    uint32_t k0[kWave], len[kWave], pre[kWave];
};

// Samples of a segment of length N whose coordinate along an axis may lie in
// [lo, hi]: [k0, k1], a float estimate of the exact window, never narrower:
// differences are exact in float, the reciprocal and two products are off by
// less than 2^-21 of a k inside the segment.
struct AxisSteps {
    int32_t p0;
    bool flat;
    float per, slack;  // samples a voxel
    __device__ __forceinline__ AxisSteps(int32_t p0_, int32_t p1, uint32_t N)
        : p0(p0_), flat(p0_ == p1), per((float)N * __builtin_amdgcn_rcpf((float)(p1 - p0_))),
          slack(0.01f + (float)N * 0x1p-20f) {}
    __device__ __forceinline__ void clip(int32_t lo, int32_t hi, float& k0, float& k1) const {
        const float a = ((float)(lo - p0) - 0.5f) * per, b = ((float)(hi - p0) + 0.5f) * per;
        const float in = lo <= p0 && p0 <= hi ? INFINITY : -INFINITY;  // (the whole axis, or none)
        k0 = fmaxf(k0, flat ? -in : fminf(a, b) - slack);
        k1 = fminf(k1, flat ? in : fmaxf(a, b) + slack);
    }
};

// A run of the volume's bits: from voxel xlo of row ylo of slab zlo to voxel xhi
// of row yhi of slab zhi.
struct SlabBox {
    int32_t zlo, zhi, ylo, yhi, xlo, xhi;
    bool one;    // inside one slab
    bool whole;  // every row of its slabs
    // Whether a segment's ranges meet it.
    __device__ __forceinline__ bool meets_y(int32_t ya, int32_t yb, int32_t za, int32_t zb) const {
        const bool first = (za <= zlo) & (yb >= ylo), last = (zb >= zhi) & (ya <= yhi);
        return one ? first & last : first | last | ((za < zhi) & (zb > zlo) & (zhi - zlo > 1));
    }
    // The segment's samples that may lie in it: from the first to the last of
    // those in its first slab, its last, and the ones between.
    __device__ __forceinline__ void window(const AxisSteps& x, const AxisSteps& y, const AxisSteps& z, float n, int32_t dy,
                                           float& k0, float& k1) const {
        float a = 0.0f, b = n;
        const bool slabs = whole && !(one && ylo == yhi);  // no more than z says
        z.clip(zlo, slabs ? zhi : zlo, a, b);
        if (slabs) {
            k0 = a;
            k1 = b;
            return;
        }
        y.clip(ylo, one ? yhi : dy - 1, a, b);
        if (one && ylo == yhi) x.clip(xlo, xhi, a, b);
        k0 = a <= b ? a : INFINITY;
        k1 = a <= b ? b : -INFINITY;
        if (one) return;
        auto also = [&](int32_t z0, int32_t z1, int32_t y1) {
            float c = 0.0f, d = n;
            z.clip(z0, z1, c, d);
            y.clip(0, y1, c, d);
            k0 = c <= d ? fminf(k0, c) : k0;
            k1 = c <= d ? fmaxf(k1, d) : k1;
        };
        also(zhi, zhi, yhi);
        if (zhi - zlo > 1) also(zlo + 1, zhi - 1, dy - 1);
    }
};

// Whether the runs are cut by the work in them (vox_slabs.h), given as differences
// in `load`, and then the boundaries w[0], w[1] of workgroup blockIdx.x's run; by
// one wave.  Every workgroup looks at the same samples and cuts alike.
__device__ __forceinline__ bool slab_cut(const uint32_t* load, uint32_t runs, uint32_t n, uint32_t samples, uint32_t nwords,
                                         uint32_t words, uint32_t* w) {
    const uint32_t lane = __lane_id();
    static_assert(kSlabMaxRuns == 8 * kWave, "eight runs a lane");
    uint32_t work[8], before[8], sum = 0, max = 0;
#pragma unroll
    for (uint32_t j = 0; j < 8u; ++j) before[j] = sum += load[8u * lane + j];
    const uint32_t first = wave_inclusive_sum_dpp(sum) - sum;
    sum = 0;
#pragma unroll
    for (uint32_t j = 0; j < 8u; ++j) {
        work[j] = 8u * lane + j < runs ? first + before[j] : 0u;
        max = work[j] > max ? work[j] : max;
        before[j] = sum;
        sum += work[j];
    }
    const uint32_t upto = wave_inclusive_sum_dpp(sum);
    const uint32_t all = __builtin_amdgcn_readlane(upto, kWave - 1);
    if (__builtin_amdgcn_ballot_w64(slab_uneven(all, max, runs, n, samples, words)) == 0) return false;
    const uint32_t base = slab_base(all, runs), total = runs * base + all;
    for (uint32_t e = 0; e < 2u; ++e) {
        const uint32_t r = blockIdx.x + e;
        if (r == runs) {
            w[e] = nwords;
            continue;
        }
        const uint32_t target = slab_target(r, runs, total);
        // The last run that begins at or before it.
        uint32_t i = 0, start = 0, own = 0;
#pragma unroll
        for (uint32_t j = 0; j < 8u; ++j) {
            const uint32_t at = (8u * lane + j) * base + (upto - sum) + before[j];
            const uint64_t m = __builtin_amdgcn_ballot_w64(8u * lane + j < runs && at <= target);
            if (m == 0) continue;
            const uint32_t l = 63u - (uint32_t)__builtin_clzll(m);
            if (8u * l + j >= i) {
                i = 8u * l + j;
                start = __builtin_amdgcn_readlane(at, l);
                own = __builtin_amdgcn_readlane(work[j], l);
            }
        }
        w[e] = slab_word(target, i, start, base + own, words, nwords);
    }
    return true;
}

// One launch for a whole small call, with no atomics on the volume and no
// clear pass: every workgroup holds a run of the volume's words in LDS, reads
// every segment, and sets the voxels that fall into its run of bits; then it
// writes the run once.  A wave tests 64 segments at a time against the run's z
// and y ranges and queues those that may touch it; from a queue of 64 it takes
// each segment's k-window in the run (every coordinate is monotone in k), cuts
// the windows into chunks of 8 samples, and its lanes take a chunk each, with one
// division per axis at its start, testing each voxel against the run.
// The runs are the same number of words each, or cut by the work in them (slab_cut)
// where the segments lie in few of them: the workgroups begin with the first while
// the last wave of each makes an estimate, and begin again with the second.  (Without
// `look` there is too little work for a cut.)
// Counts: each group of 64 segments by one workgroup.  The status word: by
// workgroup 0, which sees all segments as the others do.
//
// Bound: latency (one launch, the segments from L2, a few divisions a hit).
// Against the clear and device atomics on the volume (k_grid_direct), cleared, us a
// call: uniform end points, 1 000 segments in 256^3 7.1 / 10.4, 16 384 there
// 36 / 76, 16 384 in 512^3 47 / 164; the same in one z slice 14.2 / 20.8,
// 58 / 161 and 85 / 159 (without the cut 40, 615 and 1175, the work of one
// workgroup; the estimate costs 0.1 to 0.3 of the 7.1, and 0.6 where all waves wait
// for it); at most 8 voxels long, 16 384 in 512^3 13.3 / 11.1, and in one slice
// 18.4 / 10.2 (without the cut 92); all in 8 rows of one slice there, few units of
// words, 864 / 467, but 4 000 of them 226 / 1540.
// Windows by exact divisions, and by every lane for its own segment, hit or not:
// 74 us for 16 384 uniform ones in 256^3.
template <bool kAligned8, bool kEuclid>
__global__ __launch_bounds__(kSlabBlock) void k_grid_slabs(const int32_t* __restrict__ segs, int32_t n, int32_t dx,
                                                           int32_t dy, int32_t dz, uint32_t* __restrict__ grid,
                                                           uint32_t nwords, uint32_t words, bool clear, bool look,
                                                           int32_t* __restrict__ counts,
                                                           int32_t* __restrict__ status) {
    extern __shared__ __align__(16) uint32_t run[];
    __shared__ SlabHits hits[kSlabBlock / kWave];
    __shared__ uint32_t load[kSlabMaxRuns], bounds_s[2], cut_s;
    __shared__ int32_t bad_s;
    const uint32_t lane = __lane_id(), wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    SlabHits& h = hits[wave];
    auto inside = [&](const Seg& g) {
        return ((uint32_t)g.p0[0] < (uint32_t)dx) & ((uint32_t)g.p1[0] < (uint32_t)dx) & ((uint32_t)g.p0[1] < (uint32_t)dy) &
               ((uint32_t)g.p1[1] < (uint32_t)dy) & ((uint32_t)g.p0[2] < (uint32_t)dz) & ((uint32_t)g.p1[2] < (uint32_t)dz);
    };
    // The last wave looks at the work in each of the runs of `words` words, by
    // samples, several a lane.  (Eight neighbours at a time: whole lines; beyond the
    // last, that one again.)
    const uint32_t samples = (uint32_t)n < kSlabSamples ? (uint32_t)n : kSlabSamples;
    const bool looks = look && wave == kSlabBlock / kWave - 1;
    constexpr int kSamplesALane = kSlabSamples / kWave;
    Seg sample[kSamplesALane];
    if (looks) {
#pragma unroll
        for (int j = 0; j < kSamplesALane; ++j) {
            const uint32_t st = (uint32_t)j * kWave + lane;
            sample[j] = load_seg<kAligned8>(segs, (uint32_t)n > kSlabSamples ? st / 8u * (uint32_t)n / (kSlabSamples / 8u) + st % 8u
                                                  : st < samples ? st : samples - 1u);
        }
    }
    // Segments of a round: the last wave takes none where the others have two a lane
    // at most.  (A few more than 1 000 segments in 256^3, one round of all waves: 7.8
    // us, waiting for the wave that does both.)
    const int32_t round = look && n <= 2 * (kSlabBlock - kWave) ? kSlabBlock - kWave : kSlabBlock;
    // The thread's first two segments (beyond the last, that one again).
    auto load_at = [&](int32_t i) {
        i += (int32_t)threadIdx.x;
        return load_seg<kAligned8>(segs, i < n ? i : n - 1);
    };
    Seg sa = {}, sb = {};
    if (n > 0) {
        sa = load_at(0);
        sb = load_at(round);
    }
    const Seg own[2] = {sa, sb};
    if (threadIdx.x == 0) {
        bad_s = 0;
        cut_s = 0u;
    }
    // The run's words and, of its voxels, the first and the last.
    uint32_t w0, nw, nbits;
    SlabBox box;
    const uint32_t slab = (uint32_t)dx * (uint32_t)dy;
    auto take_run = [&](uint32_t from, uint32_t to) {
        w0 = from;
        nw = to - from;
        // (Fewer than 2^28 bits.)
        const uint32_t bits = slab * (uint32_t)dz, first = w0 * 32u;
        nbits = nw != 0u ? (first + nw * 32u < bits ? nw * 32u : bits - first) : 0u;
        const uint32_t last = nw != 0u ? first + nbits - 1u : first;
        box.zlo = (int32_t)(first / slab);
        box.ylo = (int32_t)((first - (uint32_t)box.zlo * slab) / (uint32_t)dx);
        box.xlo = (int32_t)(first - (uint32_t)box.zlo * slab - (uint32_t)box.ylo * (uint32_t)dx);
        box.zhi = (int32_t)(last / slab);
        box.yhi = (int32_t)((last - (uint32_t)box.zhi * slab) / (uint32_t)dx);
        box.xhi = (int32_t)(last - (uint32_t)box.zhi * slab - (uint32_t)box.yhi * (uint32_t)dx);
        box.one = box.zlo == box.zhi;
        box.whole = box.ylo == 0 && box.yhi == dy - 1;
        if (nw == 0u) box.zhi = -1;  // met by none
        uint4* r4 = reinterpret_cast<uint4*>(run);
        for (uint32_t u = threadIdx.x; u < (nw + 3u) / 4u; u += kSlabBlock) r4[u] = make_uint4(0u, 0u, 0u, 0u);
    };
    {
        const uint32_t first = blockIdx.x * words;
        take_run(first, nwords - first < words ? nwords : first + words);
    }
    lds_barrier();
    auto wave_fence = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    // The others begin meanwhile, and leave off when the runs are cut anew.
    if (looks) {
#pragma unroll
        for (uint32_t i = 0; i < kSlabMaxRuns / kWave; ++i) load[i * kWave + lane] = 0u;
        wave_fence();
        // A sample's work spread over the runs from one end point's to the other's.
        // (Out by one at most, and the same for every workgroup; a segment that is
        // not inside the volume counts for the runs nearest to it.)
        const float per = __builtin_amdgcn_rcpf((float)words * 32.0f), last = (float)(gridDim.x - 1u);
        auto place = [&](const int32_t* p) {
            const float row = (float)(int32_t)((uint32_t)p[2] * (uint32_t)dy + (uint32_t)p[1]);
            return fminf(fmaxf((row * (float)dx + (float)p[0]) * per, 0.0f), last);
        };
#pragma unroll
        for (int j = 0; j < kSamplesALane; ++j) {
            const Seg& g = sample[j];
            const float r0 = place(g.p0), r1 = place(g.p1);
            const uint32_t lo = (uint32_t)fminf(r0, r1), hi = (uint32_t)fmaxf(r0, r1);
            uint32_t N = 0;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const uint32_t d = (uint32_t)g.p1[a] - (uint32_t)g.p0[a];
                const int32_t m = (int32_t)d < 0 ? (int32_t)(0u - d) : (int32_t)d;
                N = (uint32_t)m > N ? (uint32_t)m : N;
            }
            const uint32_t work = (uint32_t)j * kWave + lane < samples ? slab_work(N, hi - lo + 1u) : 0u;
            atomicAdd(&load[lo], work);
            if (hi + 1u < kSlabMaxRuns) atomicAdd(&load[hi + 1u], 0u - work);
        }
        wave_fence();
        if (slab_cut(load, gridDim.x, (uint32_t)n, samples, nwords, words, bounds_s) && lane == 0)
            __hip_atomic_store(&cut_s, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    auto cut_anew = [&] { return __hip_atomic_load(&cut_s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != 0u; };

    bool first = true;  // the runs are not cut anew, or not yet
    // The voxels of the queue's segments [0, count), count <= 64.
    auto work = [&](uint32_t count) {
        uint32_t k0 = 0, len = 0;
        Seg g = {};
        if (n <= 2 * round) {  // a lane of this wave has it
            const int32_t i = (int32_t)h.queue[lane];
            const int from = i % kWave << 2;
            auto take = [&](const Seg& of, bool mine) {
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const int32_t v0 = __builtin_amdgcn_ds_bpermute(from, of.p0[a]), v1 = __builtin_amdgcn_ds_bpermute(from, of.p1[a]);
                    g.p0[a] = mine ? v0 : g.p0[a];
                    g.p1[a] = mine ? v1 : g.p1[a];
                }
            };
            take(own[0], true);
            if (n > round) take(own[1], i >= round);
        } else if (lane < count) {
            g = load_seg<kAligned8>(segs, h.queue[lane]);
        }
        if (lane < count) {
            const bool valid = inside(g);
            if (!valid) g = Seg{};
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                h.seg[a][lane] = g.p0[a];
                h.seg[3 + a][lane] = g.p1[a];
            }
            const uint32_t N = kEuclid ? euclid_length(g) : seg_axes(g).N;
            float ka = 0.0f, kb = (float)N;
            box.window(AxisSteps(g.p0[0], g.p1[0], N), AxisSteps(g.p0[1], g.p1[1], N), AxisSteps(g.p0[2], g.p1[2], N), kb, dy, ka,
                       kb);
            if (valid && ka <= kb) {
                k0 = (uint32_t)__builtin_ceilf(ka);
                const uint32_t k1 = (uint32_t)kb < N ? (uint32_t)kb : N;
                len = k1 >= k0 ? k1 - k0 + 1u : 0u;
            }
        }
        const uint32_t ch = (len + kSlabChunk - 1u) / kSlabChunk;
        const uint32_t incl = wave_inclusive_sum_dpp(ch);
        const uint32_t chunks = __builtin_amdgcn_readlane(incl, kWave - 1);
        h.k0[lane] = k0;
        h.len[lane] = len;
        h.pre[lane] = incl - ch;
        wave_fence();
        for (uint32_t q0 = 0; q0 < chunks && !(first && cut_anew()); q0 += kWave) {
            const uint32_t q = q0 + lane;
            if (q >= chunks) continue;
            // The last lane whose first chunk is at most q owns chunk q
            // (the lanes without chunks before it share its number).
            uint32_t o = 0;
#pragma unroll
            for (uint32_t step = kWave / 2; step > 0; step >>= 1) o += h.pre[o + step] <= q ? step : 0u;
            Seg s;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                s.p0[a] = h.seg[a][o];
                s.p1[a] = h.seg[3 + a][o];
            }
            const uint32_t j = (q - h.pre[o]) * kSlabChunk, k = h.k0[o] + j, left = h.len[o] - j;
            const uint32_t cnt = left < kSlabChunk ? left : kSlabChunk;
            const SegAxes ax = seg_axes(s);
            const uint32_t N = kEuclid ? euclid_length(s) : ax.N, two_n = 2u * N;
            AxisStep st[3] = {};
            if (N) axis_init3(ax.a, ax.neg, N, k, st);
            int32_t stride[3];
            int64_t at = -(int64_t)w0 * 32;
            const int32_t full[3] = {1, dx, (int32_t)slab};
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                stride[a] = ax.neg[a] ? -full[a] : full[a];
                at += (int64_t)full[a] * (ax.neg[a] ? ax.p0[a] - (int32_t)st[a].q : ax.p0[a] + (int32_t)st[a].q);
            }
            uint32_t idx = (uint32_t)at;  // mod 2^32: a bit of the run if below nbits
            for (uint32_t t = 0; t < cnt; ++t) {
                if (idx < nbits) atomicOr(&run[idx >> 5], 1u << (idx & 31u));
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    st[a].r += st[a].two_a;
                    const bool c = st[a].r >= two_n;
                    st[a].r -= c ? two_n : 0u;
                    idx += c ? (uint32_t)stride[a] : 0u;
                }
            }
        }
        wave_fence();  // the scratch is rewritten by the wave's next segments
    };

    // Counts.
    if (!kEuclid && counts) {
        for (int32_t i0 = ((int32_t)wave * (int32_t)gridDim.x + (int32_t)blockIdx.x) * kWave; i0 < n;
             i0 += kSlabBlock * (int32_t)gridDim.x) {
            const int32_t i = i0 + (int32_t)lane;
            if (i >= n) continue;
            const int64_t c = seg_length(load_seg<kAligned8>(segs, i)) + 1;
            counts[i] = (int32_t)(c > 0x7FFFFFFFll ? 0x7FFFFFFFll : c);
        }
    }
    // Every workgroup tests every segment, so an instruction here is 0.1 us of a
    // call of 16 384: few of them where no segment of 64 is near the run.
    bool bad = false;
    uint32_t queued = 0;
    auto test = [&](const Seg& g, int32_t i0) {
        if (blockIdx.x == 0) bad |= !inside(g);
        const int32_t za = g.p0[2] < g.p1[2] ? g.p0[2] : g.p1[2], zb = g.p0[2] < g.p1[2] ? g.p1[2] : g.p0[2];
        const bool near = (za <= box.zhi) & (zb >= box.zlo);
        if (__builtin_amdgcn_ballot_w64(near) == 0) return;
        const int32_t i = i0 + (int32_t)threadIdx.x;
        bool hit = near & (i < n);
        if (!box.whole) {
            const int32_t ya = g.p0[1] < g.p1[1] ? g.p0[1] : g.p1[1], yb = g.p0[1] < g.p1[1] ? g.p1[1] : g.p0[1];
            hit &= box.meets_y(ya, yb, za, zb);
        }
        const uint64_t m = __builtin_amdgcn_ballot_w64(hit);
        if (hit)
            h.queue[queued + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] =
                (uint32_t)i;
        queued += (uint32_t)__popcll(m);
    };
    const int32_t wave0 = (int32_t)wave * kWave < round ? (int32_t)wave * kWave : n;
    for (;; first = false) {
        for (int32_t i0 = 0;;) {
            for (; i0 + wave0 < n && queued < (uint32_t)kWave; i0 += 2 * round) {
                test(sa, i0);
                sa = load_at(i0 + 2 * round);
                test(sb, i0 + round);
                sb = load_at(i0 + 3 * round);
            }
            if (queued == 0 || (first && cut_anew())) break;
            wave_fence();
            const uint32_t count = queued < (uint32_t)kWave ? queued : (uint32_t)kWave;
            work(count);
            queued -= count;
            const uint32_t q0 = h.queue[kWave + lane], q1 = h.queue[2 * kWave + lane];
            wave_fence();
            h.queue[lane] = q0;
            h.queue[kWave + lane] = q1;
            wave_fence();
        }
        lds_barrier();
        if (!first || cut_s == 0u) break;
        take_run(__builtin_amdgcn_readfirstlane(bounds_s[0]), __builtin_amdgcn_readfirstlane(bounds_s[1]));
        queued = 0;
        sa = load_at(0);
        sb = load_at(round);
        lds_barrier();
    }
    if (blockIdx.x == 0 && __ballot(bad) != 0 && lane == 0) atomicOr(&bad_s, kStatusOutOfRange);
    __syncthreads();
    if (blockIdx.x == 0 && threadIdx.x == 0) *status = bad_s;
    // (words is a multiple of 32: every run but the last is whole 16-byte
    // units.)  Added to what the volume holds with atomics, as the direct
    // form does: whole lines at a time, they cost little.
    if (clear) {
        uint4* dst = reinterpret_cast<uint4*>(grid + w0);
        for (uint32_t u = threadIdx.x; u < nw / 4; u += kSlabBlock) dst[u] = reinterpret_cast<const uint4*>(run)[u];
        for (uint32_t w = nw / 4 * 4 + threadIdx.x; w < nw; w += kSlabBlock) grid[w0 + w] = run[w];
    } else {
        for (uint32_t w = threadIdx.x; w < nw; w += kSlabBlock)
            if (run[w]) atomicOr(grid + w0 + w, run[w]);
    }
}

constexpr int64_t kSlabMaxWords = 16384;
static_assert(sizeof(SlabHits) * (kSlabBlock / kWave) + (kSlabMaxRuns + 16) * 4 + (size_t)slab_room(kSlabMaxWords) * 4 <= 163840,
              "the runs fit a workgroup's LDS");

// Words of a workgroup's run: 256 runs, or runs of 64 KiB in larger volumes.
static int64_t slab_words(int64_t nwords) {
    int64_t w = ((nwords + 255) / 256 + 31) / 32 * 32;
    if (w < 64) w = 64;
    return w > kSlabMaxWords ? kSlabMaxWords : w;
}

// Which calls take the slabs.  Every workgroup reads every segment, 0.3 us a
// thousand and more (30 000 in 300 x 299 x 187, uniform / at most 8 voxels long:
// 61 / 17 us, direct 133 / 11; 16 384 in 256^3 36 / 11, direct 76 / 9), so their
// product is bounded; more than
// 512 runs (64 KiB each) lose against the direct form (1000 x 700 x 600, 4 000
// segments of log-uniform length 33 against 28 us), and so do many segments in a
// small volume, whose direct atomics are few and stay in the L2 (us, slabs /
// direct: 16 000 short ones in 96 x 86 x 87 11.9 / 8.9, 8 000 9.3 / 8.5; 16 000
// uniform ones in 64^3 26.5 / 24.4, 8 000 16.3 / 16.0, but in 128^3 26 / 38).  The
// line lies below where the two meet: 1 000 in 96^3 7.4 / 8.5, 2 000 7.6 / 8.4,
// 4 000 11.1 / 11.9.
constexpr int64_t kSlabMaxTests = int64_t(1) << 23;
constexpr int64_t kSlabSmallVolume = 65536;  // words
constexpr int64_t kSlabSmallSegments = 1536;

static bool use_slabs(int64_t n, int32_t dx, int32_t dy, int32_t dz, bool euclid, bool counts) {
    // (The Euclidean counts need whole walks; bits relative to a run, within
    // a z slab of it, are 32-bit.)
    if (euclid && counts) return false;
    if ((int64_t)dx * dy > (int64_t(1) << 28)) return false;
    const int64_t nwords = ((int64_t)dx * dy * dz + 31) / 32, w = slab_words(nwords), runs = (nwords + w - 1) / w;
    if (nwords <= kSlabSmallVolume && n > kSlabSmallSegments) return false;
    return runs <= (int64_t)kSlabMaxRuns && n * runs <= kSlabMaxTests;
}

template <bool kAligned8, bool kEuclid>
static hipError_t launch_slabs(const int32_t* segs, int64_t n, int32_t dx, int32_t dy, int32_t dz, uint32_t* grid,
                               int32_t* counts, bool clear, int32_t* status, hipStream_t stream) {
    const int64_t nwords = ((int64_t)dx * dy * dz + 31) / 32, w = slab_words(nwords);
    const unsigned wgs = (unsigned)((nwords + w - 1) / w);
    static const hipError_t attr = hipFuncSetAttribute((const void*)k_grid_slabs<kAligned8, kEuclid>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                                       (int)slab_room(kSlabMaxWords) * 4);
    if (attr != hipSuccess) return attr;
    const int32_t side = dx > dy ? (dx > dz ? dx : dz) : (dy > dz ? dy : dz);
    k_grid_slabs<kAligned8, kEuclid><<<dim3(wgs), kSlabBlock, (size_t)slab_room((uint32_t)w) * 4, stream>>>(
        segs, (int32_t)n, dx, dy, dz, grid, (uint32_t)nwords, (uint32_t)w, clear, slab_look(n, side, w), counts, status);
    return hipGetLastError();
}

// Plain calls with at most this many segments do not take the brick path, whose
// three to five launches and three passes cost 30 us with any segments at all
// (1 000 segments in 256^3: 7 against 30 us a call).  With more it depends on
// their lengths, which the host does not know: 16 384 of log-uniform length in
// 512^3 / 960^3 take 19 / 77 us here and 38 / 123 on the brick path, but uniform
// ones 47 / 308 and 42 / 136.
constexpr int64_t kDirectMaxSegments = 16384;

// The brick path serves calls with more segments than that, on volumes whose
// rows are whole words and whose piece ids fit 32 bits; everything else takes
// the direct path.
static bool use_bricks(int64_t n, int32_t dx, int32_t dy, int32_t dz, bool euclid, BrickGeom& bg, Tuning& t) {
    if (n <= kDirectMaxSegments) return false;
    if (euclid && !euclid_bricks_ok(dx, dy, dz)) return false;
    if (!tuning_cache_lookup(dx, dy, dz, n, t)) {
        default_brick_lg(dx, dy, dz, t.lg);
        t.fill_wgs_per_cu = 0;
    }
    if (!brick_geometry(dx, dy, dz, t.lg, bg)) return false;
    if (!brick_shape_supported(bg.lg)) return false;
    if (n >= (int64_t(1) << 31) - 1) return false;
    return max_pieces(n, bg) < (uint64_t(1) << 32) - 1;
}

size_t grid_workspace_bytes(int64_t n, int32_t dx, int32_t dy, int32_t dz) {
    BrickGeom bg;
    Tuning t;
    // (The Euclidean N takes the brick path under the same rules, but for the
    // volume's diagonal; the workspace bound covers both.)
    if (use_bricks(n, dx, dy, dz, false, bg, t)) return brick_workspace_bytes(n, bg);
    return kAlign;
}

size_t grid_compact_fixed_bytes(int64_t n, int32_t dx, int32_t dy, int32_t dz) {
    BrickGeom bg;
    Tuning t;
    if (!use_bricks(n, dx, dy, dz, false, bg, t)) return kAlign;
    return batch_fixed_bytes(batch_launch(1u, (uint64_t)n, bg.lg));
}

GridWork grid_workspace(void* d_work, size_t work_bytes, int64_t n, int32_t dx, int32_t dy, int32_t dz) {
    (void)n; (void)dx; (void)dy; (void)dz;
    GridWork w;
    w.status = static_cast<int32_t*>(d_work);
    w.bytes = work_bytes;
    return w;
}

hipError_t launch_grid(const int32_t* segs, int64_t n, bool aligned8, int32_t dx, int32_t dy,
                       int32_t dz, uint32_t* grid, int32_t* counts, uint32_t flags,
                       const GridWork& w, hipStream_t stream) {
    BrickGeom bg;
    Tuning t;
    // The brick path reads segments with 8-byte loads; arrays that are only
    // 4-byte aligned take the direct path.
    const bool euclid = (flags & 2u) != 0;  // VOX_GRID_EUCLID
    if (aligned8 && use_bricks(n, dx, dy, dz, euclid, bg, t)) {
        vox_scene one{};
        one.segs = reinterpret_cast<const vox_segment*>(segs);
        one.n = n;
        one.dim_x = dx;
        one.dim_y = dy;
        one.dim_z = dz;
        one.flags = flags & 3u;
        one.grid = grid;
        one.counts = counts;
        // A workspace below the worst case of records: the call runs as a
        // one-scene batch, whose direct kernels serve it when its records do
        // not fit.
        const BrickLaunch L = w.bytes >= brick_workspace_bytes(n, bg) ? plain_launch(n, bg)
                                                                       : batch_launch(1u, (uint64_t)n, bg.lg);
        return launch_bricks(nullptr, &one, L, t.fill_wgs_per_cu, w.status, w.bytes, stream);
    }
    hipError_t e = hipSuccess;
    const int64_t nwords = ((int64_t)dx * dy * dz + 31) / 32;
    if (use_slabs(n, dx, dy, dz, euclid, counts != nullptr)) {
        KernelTimer timer("grid_slabs", stream);
        const bool clear = (flags & 1u) != 0;
        if (euclid)
            return aligned8 ? launch_slabs<true, true>(segs, n, dx, dy, dz, grid, counts, clear, w.status, stream)
                            : launch_slabs<false, true>(segs, n, dx, dy, dz, grid, counts, clear, w.status, stream);
        return aligned8 ? launch_slabs<true, false>(segs, n, dx, dy, dz, grid, counts, clear, w.status, stream)
                        : launch_slabs<false, false>(segs, n, dx, dy, dz, grid, counts, clear, w.status, stream);
    }
    if (flags & 1u) {
        int64_t blocks = (nwords / 4 + kGridBlock - 1) / kGridBlock;
        if (blocks > 8192) blocks = 8192;
        if (blocks < 1) blocks = 1;
        KernelTimer timer("grid_clear", stream);
        k_grid_clear<<<dim3((unsigned)blocks), kGridBlock, 0, stream>>>(grid, nwords, w.status);
    } else {
        KernelTimer timer("grid_init", stream);
        k_grid_init<<<1, 64, 0, stream>>>(w.status);
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (n == 0) return hipSuccess;
    constexpr int kSegsPerBlock = kGridBlock / kSampleLanes;
    int64_t blocks = (n + kSegsPerBlock - 1) / kSegsPerBlock;
    if (blocks > 16384) blocks = 16384;
    dim3 gridDim((unsigned)blocks);
    KernelTimer timer(euclid ? "grid_direct_euclid" : "grid_direct", stream);
    auto direct = [&](auto a8, auto eu) {
        constexpr bool kA8 = decltype(a8)::value, kEu = decltype(eu)::value;
        if (direct_runs(n, nwords))
            k_grid_direct<kA8, kEu, true><<<gridDim, kGridBlock, 0, stream>>>(segs, n, dx, dy, dz, grid, counts,
                                                                              w.status);
        else
            k_grid_direct<kA8, kEu, false><<<gridDim, kGridBlock, 0, stream>>>(segs, n, dx, dy, dz, grid, counts,
                                                                               w.status);
    };
    if (euclid) {
        if (aligned8)
            direct(std::true_type{}, std::true_type{});
        else
            direct(std::false_type{}, std::true_type{});
    } else {
        if (aligned8)
            direct(std::true_type{}, std::false_type{});
        else
            direct(std::false_type{}, std::false_type{});
    }
    return hipGetLastError();
}

}  // namespace vox
