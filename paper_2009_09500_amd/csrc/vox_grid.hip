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

// A wave's segments that may hold voxels of its run (a queue of up to 128),
// and the windows of the 64 it works on.
struct SlabHits {
    int32_t seg[6][2 * kWave];
    uint32_t k0[kWave], len[kWave], pre[kWave];
};

// Samples of a segment of length N whose coordinate along an axis may lie in
// [lo, hi]: [k0, k1], a float estimate of the exact window, never narrower:
// differences are exact in float, the reciprocal and two products are off by
// less than 2^-21 of a k inside the segment.
__device__ __forceinline__ void axis_window_about(int32_t p0, int32_t p1, uint32_t N, int32_t lo, int32_t hi,
                                                  float& k0, float& k1) {
    if (p0 == p1) return;
    const float per = (float)N * __builtin_amdgcn_rcpf((float)(p1 - p0));
    const float a = ((float)(lo - p0) - 0.5f) * per, b = ((float)(hi - p0) + 0.5f) * per;
    const float slack = 0.01f + (float)N * 0x1p-20f;
    k0 = fmaxf(k0, fminf(a, b) - slack);
    k1 = fminf(k1, fmaxf(a, b) + slack);
}

// One launch for a whole small call, with no atomics on the volume and no
// clear pass: workgroup b holds words [b * words, (b + 1) * words) of the volume
// in LDS, reads every segment, and sets the voxels that fall into its run of
// bits; then it writes the run once.  A wave tests 64 segments at a time
// against the run's z (and, for a run inside one z slab, y) range and queues
// those that may touch it; from a queue of 64 it takes each segment's k-window
// in that range (every coordinate is monotone in k), cuts the windows into
// chunks of 8 samples, and its lanes take a chunk each, with one division per
// axis at its start, testing each voxel against the run.
// Counts: each group of 64 segments by one workgroup.  The status word: by
// workgroup 0, which sees all segments as the others do.
//
// Bound: latency (one launch, the segments from L2, a few divisions a hit).
// Against the clear and one device atomic a voxel (25 G a second), uniform end
// points, cleared: 1 000 segments in 256^3 11.3 -> 7.8 us a call, 16 384 there
// 85 -> 40 us, 16 384 in 512^3 182 -> 50 us.  Windows by exact divisions, and
// by every lane for its own segment, hit or not: 74 us for 16 384 in 256^3.
template <bool kAligned8, bool kEuclid>
__global__ __launch_bounds__(kSlabBlock) void k_grid_slabs(const int32_t* __restrict__ segs, int32_t n, int32_t dx,
                                                           int32_t dy, int32_t dz, uint32_t* __restrict__ grid,
                                                           int64_t nwords, uint32_t words, bool clear,
                                                           int32_t* __restrict__ counts,
                                                           int32_t* __restrict__ status) {
    extern __shared__ __align__(16) uint32_t run[];
    __shared__ SlabHits hits[kSlabBlock / kWave];
    __shared__ int32_t bad_s;
    const uint32_t lane = __lane_id(), wave = threadIdx.x / kWave;
    SlabHits& h = hits[wave];
    const int64_t w0 = (int64_t)blockIdx.x * words;
    const uint32_t nw = nwords - w0 < (int64_t)words ? (uint32_t)(nwords - w0) : words;
    const int64_t slab = (int64_t)dx * dy, b0 = w0 * 32;
    const int64_t total = slab * dz;
    const int64_t b1 = b0 + (int64_t)nw * 32 < total ? b0 + (int64_t)nw * 32 : total;
    const uint32_t nbits = (uint32_t)(b1 - b0);
    // Voxels of the run: z in [zlo, zhi], y in [ylo, yhi].
    const int32_t zlo = (int32_t)(b0 / slab), zhi = (int32_t)((b1 - 1) / slab);
    const int32_t ylo = zlo == zhi ? (int32_t)((b0 - zlo * slab) / dx) : 0;
    const int32_t yhi = zlo == zhi ? (int32_t)((b1 - 1 - zlo * slab) / dx) : dy - 1;
    for (uint32_t w = threadIdx.x; w < nw; w += kSlabBlock) run[w] = 0u;
    if (threadIdx.x == 0) bad_s = 0;
    __syncthreads();

    auto wave_fence = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    // The voxels of the queue's segments [0, count), count <= 64.
    auto work = [&](uint32_t count) {
        uint32_t k0 = 0, len = 0;
        if (lane < count) {
            Seg g;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                g.p0[a] = h.seg[a][lane];
                g.p1[a] = h.seg[3 + a][lane];
            }
            const uint32_t N = kEuclid ? euclid_length(g) : (uint32_t)seg_length(g);
            float ka = 0.0f, kb = (float)N;
            axis_window_about(g.p0[2], g.p1[2], N, zlo, zhi, ka, kb);
            if (zlo == zhi) axis_window_about(g.p0[1], g.p1[1], N, ylo, yhi, ka, kb);
            if (ka <= kb) {
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
        for (uint32_t q0 = 0; q0 < chunks; q0 += kWave) {
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
            int64_t at = -b0;
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

    bool bad = false;
    uint32_t queued = 0;
    Seg next = {};
    if ((int32_t)(wave * kWave + lane) < n) next = load_seg<kAligned8>(segs, wave * kWave + lane);
    for (int32_t i0 = (int32_t)wave * kWave; i0 < n; i0 += kSlabBlock) {
        const int32_t i = i0 + (int32_t)lane;
        const Seg g = next;
        if (i + kSlabBlock < n) next = load_seg<kAligned8>(segs, i + kSlabBlock);
        bool hit = false;
        if (i < n) {
            bool ok = true;
            const int32_t dim[3] = {dx, dy, dz};
#pragma unroll
            for (int a = 0; a < 3; ++a)
                ok &= (g.p0[a] >= 0) & (g.p0[a] < dim[a]) & (g.p1[a] >= 0) & (g.p1[a] < dim[a]);
            bad |= !ok;
            if (!kEuclid && counts && (uint32_t)(i0 / kWave) % gridDim.x == blockIdx.x) {
                const int64_t c = seg_length(g) + 1;
                counts[i] = (int32_t)(c > 0x7FFFFFFFll ? 0x7FFFFFFFll : c);
            }
            const int32_t za = g.p0[2] < g.p1[2] ? g.p0[2] : g.p1[2], zb = g.p0[2] < g.p1[2] ? g.p1[2] : g.p0[2];
            const int32_t ya = g.p0[1] < g.p1[1] ? g.p0[1] : g.p1[1], yb = g.p0[1] < g.p1[1] ? g.p1[1] : g.p0[1];
            hit = ok && za <= zhi && zb >= zlo && ya <= yhi && yb >= ylo;
        }
        const uint64_t m = __ballot(hit);
        if (m == 0) continue;
        if (hit) {
            const uint32_t at = queued + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                                    __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                h.seg[a][at] = g.p0[a];
                h.seg[3 + a][at] = g.p1[a];
            }
        }
        queued += (uint32_t)__popcll(m);
        wave_fence();
        if (queued >= (uint32_t)kWave) {
            work(kWave);
            queued -= kWave;
            if (lane < queued) {
#pragma unroll
                for (int a = 0; a < 6; ++a) h.seg[a][lane] = h.seg[a][kWave + lane];
            }
            wave_fence();
        }
    }
    if (queued) work(queued);
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

// Words of a workgroup's run: 256 runs, or runs of 64 KiB in larger volumes.
static int64_t slab_words(int64_t nwords) {
    int64_t w = ((nwords + 255) / 256 + 31) / 32 * 32;
    if (w < 64) w = 64;
    return w > 16384 ? 16384 : w;
}

// Which calls take the slabs.  Every workgroup reads every segment, about
// 1 us a thousand (16 384 segments of log-uniform length: 17 us in 256 runs,
// 20 us in 512; direct 22 and 44 us), so their product is bounded; more than
// 512 runs (64 KiB each) lose against the direct form (1000 x 700 x 600, 4 000
// short segments 33 against 28 us), and so do more than some segments in a small
// volume, whose direct atomics are few and stay in the L2 (96^3, uniform ones:
// 1 000 6.9 against 8.6 us, 2 000 10.3 / 8.4, 4 000 16.0 / 12.4; of log-uniform
// length 6.5 / 8.3, 7.2 / 8.3, 8.3 / 8.5).
constexpr int64_t kSlabMaxTests = int64_t(1) << 23;
constexpr int64_t kSlabMaxRuns = 512;
constexpr int64_t kSlabSmallVolume = 65536;  // words
constexpr int64_t kSlabSmallSegments = 1536;

static bool use_slabs(int64_t n, int32_t dx, int32_t dy, int32_t dz, bool euclid, bool counts) {
    // (The Euclidean counts need whole walks; bits relative to a run, within
    // a z slab of it, are 32-bit.)
    if (euclid && counts) return false;
    if ((int64_t)dx * dy > (int64_t(1) << 28)) return false;
    const int64_t nwords = ((int64_t)dx * dy * dz + 31) / 32, w = slab_words(nwords), runs = (nwords + w - 1) / w;
    if (nwords <= kSlabSmallVolume && n > kSlabSmallSegments) return false;
    return runs <= kSlabMaxRuns && n * runs <= kSlabMaxTests;
}

template <bool kAligned8, bool kEuclid>
static hipError_t launch_slabs(const int32_t* segs, int64_t n, int32_t dx, int32_t dy, int32_t dz, uint32_t* grid,
                               int32_t* counts, bool clear, int32_t* status, hipStream_t stream) {
    const int64_t nwords = ((int64_t)dx * dy * dz + 31) / 32, w = slab_words(nwords);
    const unsigned wgs = (unsigned)((nwords + w - 1) / w);
    static const hipError_t attr = hipFuncSetAttribute((const void*)k_grid_slabs<kAligned8, kEuclid>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, 16384 * 4);
    if (attr != hipSuccess) return attr;
    k_grid_slabs<kAligned8, kEuclid><<<dim3(wgs), kSlabBlock, (size_t)w * 4, stream>>>(
        segs, (int32_t)n, dx, dy, dz, grid, nwords, (uint32_t)w, clear, counts, status);
    return hipGetLastError();
}

// Plain calls with at most this many segments do not take the brick path, whose
// three to five launches and three passes cost 30 us with any segments at all
// (1 000 segments in 256^3: 7 against 30 us a call).  With more it depends on
// their lengths, which the host does not know: 16 384 of log-uniform length in
// 512^3 / 960^3 take 20 / 77 us here and 38 / 122 on the brick path, but uniform
// ones 48 / 312 and 42 / 133.
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
