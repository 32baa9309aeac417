// Bit-volume output through LDS bricks.
//
// The volume is cut into bricks of BX x BY x BZ voxels (powers of two, BX a
// multiple of 32 so brick rows are whole 32-bit words).  A brick's bits fit in
// one workgroup's LDS; the workgroup that owns a brick sets all of its voxels
// there and then writes the brick to HBM once with plain stores, which also
// clears it (no separate clear pass, no global atomics).
//
// Each segment is cut into pieces, one per brick it passes through.  As every
// coordinate of eq. (3) is monotone in k, the voxels of a segment inside one
// brick form a single k-interval, and the brick changes exactly when one
// coordinate crosses a brick boundary (exact helpers in vox_exact.h).
//
// Every kernel reads its volumes from a scene table (BrickTable followed by
// BrickScene entries) that the plan kernel writes into the workspace from
// the caller's vox_scene entries: a plain call is a table of one scene, a
// batch a table of many, whose bricks and histogram rows are numbered
// globally so that each kernel below is still one launch for the whole batch.
//
// Pipeline (one stream, no host synchronisation, no allocation):
//   plan      checks every scene, decides brick or direct kernels per scene,
//             numbers rows and bricks (block scans), writes the table, the
//             status word and the fill's work queues
//   hist      (batches) finds its row's scene and notes it for the row and
//             the bricks;
//             per segment: count N+1, range check, walk its bricks and count
//             pieces per brick in an LDS histogram; one histogram row per
//             workgroup
//   colscan   per brick, exclusive prefix of the rows over workgroups, and
//             the brick's piece total
//   base      exclusive scan of the brick totals -> bin offsets; if the
//             records do not fit the workspace, the direct kernel takes over;
//             the fill's work items: one per brick, several for a brick with
//             more than a fair share of the records
//             (a plain call of few bricks and rows: colscan and base are done
//             inside the scatter)
//   scatter   zeroes the bricks cut into several items in cleared volumes,
//             then the same walk again, writing one 16-byte piece record
//             (start point, direction, k-window in the brick) into the
//             brick's bin
//   fill      zeroes the volumes of the cleared direct scenes (batches);
//             persistent workgroups take work items from work-stealing
//             queues, set the bits of every piece with LDS atomic OR and
//             flush the brick to the volume (an item that holds part of a
//             brick with device atomic OR)
//   direct    (batches) one device atomic per voxel, for the scenes the
//             bricks do not serve
#include <type_traits>

#include "vox.h"
#include "vox_device.h"
#include "vox_direct.h"
#include "vox_exact.h"
#include "vox_internal.h"

namespace vox {

// Block-wide exclusive sum like block_exclusive_sum, synchronised with
// lds_barrier so that outstanding global loads are not waited for.
template <int kBlock>
__device__ __forceinline__ uint32_t block_exclusive_sum_lds(uint32_t v, uint32_t* lds, uint32_t& total) {
    constexpr int kWaves = kBlock / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    const int w = threadIdx.x / kWave;
    const uint32_t incl = wave_inclusive_sum(v);
    if (lane == kWave - 1) lds[w] = incl;
    lds_barrier();
    uint32_t pre = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < kWaves; ++i) {
        const uint32_t x = lds[i];
        pre += (i < w) ? x : 0u;
        tot += x;
    }
    lds_barrier();
    total = tot;
    return pre + incl - v;
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// Global-memory views: volume pointers come from the scene table, so the
// compiler cannot infer their address space; without these casts it emits
// flat stores, which also count against the LDS wait counter.
typedef __attribute__((address_space(1))) u32x4 global_u32x4;
typedef __attribute__((address_space(1))) uint32_t global_u32;

// A value that an earlier kernel wrote and that is the same for the whole
// wave, by scalar loads: the compiler cannot see that nothing in this kernel
// writes it, and would take vector loads, whose wait is also one for every
// vector load and store before them.
template <typename T>
__device__ __forceinline__ T load_uniform(const T* p) {
    typedef __attribute__((address_space(4))) const uint32_t const_u32;
    static_assert(sizeof(T) % 4 == 0, "whole words");
    const_u32* c = (const_u32*)(uintptr_t)p;
    uint32_t w[sizeof(T) / 4];
#pragma unroll
    for (unsigned i = 0; i < sizeof(T) / 4; ++i) w[i] = c[i];
    T v;
    __builtin_memcpy(&v, w, sizeof(T));
    return v;
}

typedef int16_t i16x2 __attribute__((ext_vector_type(2)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

// ------------------------------------------------------------------ kernels

__host__ __device__ constexpr uint64_t up256(uint64_t v) { return (v + 255u) & ~uint64_t(255); }

// Piece record (16 bytes): the stepping state of a piece at its first voxel
// (k = klo), made by the scatter, which has the segment at hand, so that the
// fill only unpacks it and never gathers segments.  Minor axes a < b in axis
// order, m the dominant axis (the first of the longest ones), fractions and
// slopes of the minor axes in 23 bits (fix23_fraction, fix23_slope):
//   e  fraction of a << 9 | slope of b, bits 0-8
//   t  fraction of b << 9 | slope of b, bits 9-17
//   v  slope of a << 9 | negm << 5 | slope of b, bits 18-22
//   w  the bit index of the voxel at klo inside the brick
//      | (voxels - 1) << (log2 of the brick's voxel count)
//      | m << 28 | nega << 30 | negb << 31
// Three axes need more bits, so a record of a Euclidean scene holds the
// integers (piece_record_euclid).
struct Piece {
    uint32_t e, t, v, w;
};
static_assert(sizeof(Piece) == 16, "16-byte piece records");

// Sections of the workspace: the header words, the table the plan kernel
// writes at kWorkTable, then at the table's data_off the histograms, the
// brick totals, the bin offsets, the fill's work items and the piece records
// (the rest of the workspace).
//
// Bytes from the table's data_off to the piece records.
__host__ __device__ inline uint64_t brick_data_bytes(uint64_t hist_words, uint64_t bricks) {
    return up256(hist_words * 4u) + up256(bricks * 4u) + 2u * up256((bricks + 1u) * 4u) +
           up256((bricks + kMaxExtraItems) * 4u) + up256((uint64_t)kMaxExtraItems * 4u);
}

struct WorkView {
    int32_t* status;
    uint32_t* counter;   // [kXcds] work queues of the fill, one per XCD
    uint32_t* ok;
    uint32_t* direct_all;
    uint64_t* pieces;
    uint32_t* hist;
    uint32_t* totals;
    uint32_t* bin_base;
    uint32_t* n_items;     // fill work items (header word)
    uint32_t* n_split;     // bricks cut into several items (header word)
    uint32_t* item_base;   // [bricks + 1] first extra item of each brick
    uint32_t* item_brick;  // [bricks + kMaxExtraItems] brick of each extra item
    uint32_t* split;       // [kMaxExtraItems] the bricks cut into several items
    Piece* recs;
    uint64_t rec_off;    // byte offset of the records
};

__host__ __device__ inline WorkView work_view(uint8_t* work, uint64_t data_off, uint64_t hist_words,
                                              uint32_t bricks) {
    WorkView v;
    uint32_t* w = reinterpret_cast<uint32_t*>(work);
    v.status = reinterpret_cast<int32_t*>(work) + kWStatus;
    v.counter = w + kWQueues;
    v.ok = w + kWOk;
    v.direct_all = w + kWDirectAll;
    v.pieces = reinterpret_cast<uint64_t*>(w + kWPieces);
    v.n_items = w + kWItems;
    v.n_split = w + kWSplit;
    uint64_t off = data_off;
    v.hist = reinterpret_cast<uint32_t*>(work + off);
    off += up256(hist_words * 4u);
    v.totals = reinterpret_cast<uint32_t*>(work + off);
    off += up256((uint64_t)bricks * 4u);
    v.bin_base = reinterpret_cast<uint32_t*>(work + off);
    off += up256(((uint64_t)bricks + 1u) * 4u);
    v.item_base = reinterpret_cast<uint32_t*>(work + off);
    off += up256(((uint64_t)bricks + 1u) * 4u);
    v.item_brick = reinterpret_cast<uint32_t*>(work + off);
    off += up256(((uint64_t)bricks + kMaxExtraItems) * 4u);
    v.split = reinterpret_cast<uint32_t*>(work + off);
    off += up256((uint64_t)kMaxExtraItems * 4u);
    v.recs = reinterpret_cast<Piece*>(work + off);
    v.rec_off = off;
    return v;
}

// The scene table as the kernels see it.
struct TableView {
    BrickTable h;
    const BrickScene* scenes;
    const uint32_t* direct;       // the direct scenes, in order
    const uint32_t* row_scene;    // null with one scene
    const uint32_t* brick_scene;  // null with one scene
};

__host__ __device__ __forceinline__ TableView table_view(const uint8_t* table) {
    TableView v;
    v.h = *reinterpret_cast<const BrickTable*>(table);
    v.scenes = reinterpret_cast<const BrickScene*>(table + kTableScenes);
    v.direct = reinterpret_cast<const uint32_t*>(v.scenes + v.h.n_scenes);
    if (v.h.n_scenes > 1) {
        v.row_scene = v.direct + v.h.n_scenes;
        v.brick_scene = v.row_scene + v.h.row_cap;
    } else {
        v.row_scene = v.brick_scene = nullptr;
    }
    return v;
}

__device__ __forceinline__ WorkView work_of(uint8_t* work, const TableView& tv) {
    return work_view(work, tv.h.data_off, tv.h.hist_words, tv.h.bricks);
}

// Work queues of the fill.  The 8 XCDs of the chip each have their own L2;
// workgroup w runs on XCD w % 8.  The queues deal units of one work item, or
// of two (items 2u and 2u + 1) when there are many: groups of 8 consecutive
// items (bricks along x, the fastest brick axis) go to the XCDs in turn, so
// neighbouring bricks, whose row pieces share memory lines, are flushed
// through the same L2.  A workgroup takes from its own XCD's queue first and
// then from the others.
constexpr int kXcds = 8;

struct FillQueue {
    uint32_t* counter;  // [kXcds]
    uint32_t items;     // work items in all
    uint32_t extra;     // of them extra items, rounded up to even (items [0, extra))
    uint32_t units;     // queue units
    uint32_t lg;        // log2 of the units in a group of 8 items
    bool cut;           // some brick is cut into several items
    uint32_t xcd;       // this workgroup's queue
    uint32_t wgs;       // workgroups of the launch
};

// Unit of the c-th claim on queue x.
__device__ __forceinline__ uint32_t queue_unit(uint32_t x, uint32_t c, uint32_t lg) {
    return ((c >> lg) << (lg + 3u)) + (x << lg) + (c & ((1u << lg) - 1u));
}
static_assert(kXcds == 8, "groups are dealt to 8 queues");

// A workgroup's first unit is its own by its number (no atomic); the claims
// of a queue start after those.
__device__ __forceinline__ uint32_t queue_start(const FillQueue& q, uint32_t x) {
    return (q.wgs - x + (uint32_t)kXcds - 1u) / (uint32_t)kXcds;  // workgroups x, x + 8, ... (x < wgs or 0)
}

// The next unit of this workgroup (claimed by one whole wave), or q.units
// when none is left.  A device-scope atomic costs a full memory round trip,
// so once its own queue is empty a workgroup reads all the other counters at
// once, a lane each (one round trip), and claims only from queues that still
// hold units, rather than trying each in turn; it stops when every queue is
// empty (counters only grow, so every pass either claims or finds fewer
// queues open).
__device__ __forceinline__ uint32_t claim_unit(const FillQueue& q) {
    const uint32_t lane = __lane_id(), x = lane % (uint32_t)kXcds;
    auto take = [&](uint32_t queue) {
        uint32_t c = 0;
        if (lane == 0) c = atomicAdd(&q.counter[queue], 1u);
        return queue_unit(queue, queue_start(q, queue) + (uint32_t)__builtin_amdgcn_readfirstlane(c), q.lg);
    };
    if (queue_unit(q.xcd, queue_start(q, q.xcd), q.lg) < q.units) {
        const uint32_t g = take(q.xcd);
        if (g < q.units) return g;
    }
    // (With no more units than workgroups there is nothing to claim.)
    uint64_t open = __ballot(queue_unit(x, queue_start(q, x), q.lg) < q.units);
    while (open) {
        const uint32_t c = __hip_atomic_load(&q.counter[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        open = __ballot(lane < (uint32_t)kXcds && x != q.xcd && queue_unit(x, queue_start(q, x) + c, q.lg) < q.units);
        for (uint64_t m = open; m; m &= m - 1) {
            const uint32_t g = take((uint32_t)__builtin_ctzll(m));
            if (g < q.units) return g;
        }
    }
    return q.units;
}

// The next work item of a workgroup (claimed by one whole wave): its brick (NB
// when none is left), its part [lo, hi) of the brick's records and whether
// the brick is cut into several items.  The extra items of cut bricks (their
// parts 1, 2, ...) come first, then every brick (whole, or its part 0).
// `second` holds the second item of a claimed unit of two.
struct ItemClaim {
    uint32_t brick, lo, hi, split;
};
__device__ __forceinline__ ItemClaim item_at(const WorkView& wv, const FillQueue& q, uint32_t i) {
    ItemClaim c;
    c.split = 0u;
    if (!q.cut) {  // the items are the bricks
        c.brick = i;
        c.lo = load_uniform(wv.bin_base + i);
        c.hi = load_uniform(wv.bin_base + i + 1);
        return c;
    }
    const uint32_t b = i < q.extra ? load_uniform(wv.item_brick + i) : i - q.extra;
    const uint32_t x0 = load_uniform(wv.item_base + b), k = load_uniform(wv.item_base + b + 1) - x0 + 1u;
    const uint32_t lo = load_uniform(wv.bin_base + b);
    c.brick = b;
    item_range(lo, load_uniform(wv.bin_base + b + 1) - lo, i < q.extra ? i - x0 + 1u : 0u, k, c.lo, c.hi);
    c.split = k > 1u ? 1u : 0u;
    return c;
}
__device__ __forceinline__ ItemClaim claim_item(const WorkView& wv, const FillQueue& q, uint32_t NB,
                                                uint32_t& second, bool first = false) {
    uint32_t i;
    do {
        i = second;
        second = q.items;
        if (i >= q.items) {
            uint32_t u = first ? queue_unit(q.xcd, blockIdx.x / (uint32_t)kXcds, q.lg) : q.units;
            first = false;
            if (u >= q.units) u = claim_unit(q);
            if (u >= q.units) return {NB, 0u, 0u, 0u};
            i = u;
            if (q.lg == 2u) {
                i = 2u * u;
                second = i + 1u;
            }
        }
    } while (i < q.extra && i >= load_uniform(wv.item_base + NB));  // (the rounding up)
    return item_at(wv, q, i);
}

// Histogram row of workgroup w out of G.  Each XCD takes a contiguous block
// of rows (workgroup w runs on XCD w % 8): a bin holds the records of row 0,
// then row 1, ..., so the scatter's short per-row runs of one bin that share
// memory lines are written through one L2 at about the same time.
__device__ __forceinline__ uint32_t xcd_row(uint32_t w, uint32_t G) {
    const uint32_t x = w % kXcds, a = w / kXcds;
    uint32_t start = 0;
    for (uint32_t i = 0; i < x; ++i) start += (G - i + kXcds - 1) / kXcds;  // rows of XCD i
    return start + a;
}

// The table header, status word, flags and work queues of a launch whose
// scenes have been numbered (one lane).
__device__ __forceinline__ void write_table(uint8_t* work, const BrickLaunch& L, uint64_t work_bytes, uint32_t rows_c,
                                            uint32_t bricks_c, uint32_t direct_c, uint64_t hist_c,
                                            uint64_t segs_c, uint64_t dsegs_c, bool bad) {
    uint8_t* tb = work + kWorkTable;
    BrickTable t{};
    t.magic = kTableMagic;
    t.n_scenes = L.n_scenes;
    t.rows = rows_c;
    t.bricks = bricks_c;
    for (int a = 0; a < 3; ++a) t.lg[a] = L.lg[a];
    t.hist_words = hist_c;
    t.data_off = kWorkTable + L.table_bytes;
    t.n_direct = direct_c;
    t.row_cap = L.rows;
    t.direct_segs = dsegs_c;
    *reinterpret_cast<BrickTable*>(tb) = t;
    const bool fits = segs_c <= L.total_segments && rows_c <= L.rows && bricks_c <= L.bricks;
    const WorkView wv = work_view(work, t.data_off, t.hist_words, t.bricks);
    const bool room = wv.rec_off <= work_bytes;
    uint32_t* w = reinterpret_cast<uint32_t*>(work);
    const int32_t st = bad ? kStatusInvalid : (fits ? 0 : kStatusLaunch);
    w[kWStatus] = (uint32_t)st;
    w[kWOk] = (st == 0 && room && bricks_c > 0) ? 1u : 0u;
    w[kWDirectAll] = room ? 0u : 1u;
    for (int x = 0; x < kXcds; ++x) w[kWQueues + x] = 0u;
    *wv.pieces = 0;
}

// The plan of a batch: one block reads the caller's scenes (the device
// vox_scene array), checks each against the argument rules, decides which
// scenes the brick kernels serve (8-byte-aligned segment arrays, volumes the
// bricks cover; with the Euclidean N, a diagonal below 16385) and which the
// direct kernels serve, numbers the histogram rows and bricks of all brick
// scenes (block scans), and writes the table, the status word, the brick
// queues and the flags.  A scene that breaks a rule, or scenes beyond the
// launch bounds, stop the whole call (nothing is written).  When the
// histograms and brick offsets do not fit the workspace, the direct kernels
// serve every scene.
template <int kBlock>
__global__ __launch_bounds__(kBlock) void k_brick_plan(const vox_scene* __restrict__ scenes, BrickLaunch L,
                                                           uint8_t* __restrict__ work, uint64_t work_bytes) {
    __shared__ uint32_t scan32[kBlock / kWave];
    __shared__ uint64_t scan64[kBlock / kWave];
    __shared__ uint32_t bad_s;
    uint8_t* tb = work + kWorkTable;
    BrickScene* out = reinterpret_cast<BrickScene*>(tb + kTableScenes);
    uint32_t* direct = reinterpret_cast<uint32_t*>(out + L.n_scenes);
    if (threadIdx.x == 0) bad_s = 0;
    __syncthreads();
    uint32_t rows_c = 0, bricks_c = 0, direct_c = 0;
    uint64_t hist_c = 0, segs_c = 0, dsegs_c = 0;
    for (uint32_t c0 = 0; c0 < L.n_scenes; c0 += kBlock) {
        const uint32_t i = c0 + threadIdx.x;
        BrickScene b{};
        uint32_t rows = 0, nb = 0, isd = 0;
        uint64_t hist = 0, n = 0;
        if (i < L.n_scenes) {
            const vox_scene in = scenes[i];
            if (!plan_scene(in, L.lg, L.segs_per_row, b)) atomicOr(&bad_s, 1u);
            isd = (b.flags & kSceneDirect) ? 1u : 0u;
            rows = b.rows;
            // Brick numbers of a scene start even (an odd count is rounded
            // up by a brick outside the volume, with no records), so that
            // the fill's units of two hold bricks side by side.
            nb = isd ? 0u : (b.bg.nbricks + 1u) & ~1u;
            hist = (uint64_t)rows * b.bg.nbricks;
            n = b.n > 0 ? (uint64_t)b.n : 0u;
        }
        uint32_t t_rows, t_nb, t_d;
        uint64_t t_hist, t_n, t_dn;
        const uint32_t x_rows = block_exclusive_sum<kBlock>(rows, scan32, t_rows);
        const uint32_t x_nb = block_exclusive_sum<kBlock>(nb, scan32, t_nb);
        const uint32_t x_d = block_exclusive_sum<kBlock>(isd, scan32, t_d);
        const uint64_t x_hist = block_exclusive_sum<kBlock>(hist, scan64, t_hist);
        (void)block_exclusive_sum<kBlock>(n, scan64, t_n);
        (void)block_exclusive_sum<kBlock>(isd ? n : 0u, scan64, t_dn);
        if (i < L.n_scenes) {
            b.row_base = rows_c + x_rows;
            b.brick_base = bricks_c + x_nb;
            b.hist_off = hist_c + x_hist;
            out[i] = b;
            if (isd) direct[direct_c + x_d] = i;
        }
        rows_c += t_rows;
        bricks_c += t_nb;
        direct_c += t_d;
        hist_c += t_hist;
        segs_c += t_n;
        dsegs_c += t_dn;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    write_table(work, L, work_bytes, rows_c, bricks_c, direct_c, hist_c, segs_c, dsegs_c, bad_s != 0);
}

// The scene of histogram row r of a batch: the last one whose rows start at or
// before it (direct scenes have none), by a search of 64 scenes at a time.  All
// lanes of a wave take part.
__device__ __forceinline__ uint32_t scene_of_row(const TableView& tv, uint32_t r) {
    uint32_t at = 0, len = tv.h.n_scenes;
    while (len > 1u) {
        const uint32_t step = (len + kWave - 1u) / kWave, i = at + step * __lane_id();
        const bool below = i < tv.h.n_scenes && tv.scenes[i].row_base <= r;
        at += step * ((uint32_t)__popcll(__builtin_amdgcn_ballot_w64(below)) - 1u);
        len = step;
    }
    return at;
}

// Segment range of histogram/scatter workgroup g.
__device__ __forceinline__ void seg_range(int64_t n, int g, int G, int64_t& lo, int64_t& hi) {
    int64_t per = (n + G - 1) / G;
    lo = (int64_t)g * per;
    hi = lo + per < n ? lo + per : n;
}

// A segment staged in LDS for the walk: end points as uint16 (every brick
// volume side is <= 16384).
struct StagedSeg {
    uint16_t p0[3];
    uint16_t p1[3];
};

constexpr int kStage = 4096;      // segments staged per round
constexpr int kStageBig = 8192;   // ... by the histogram when its counters leave room
constexpr uint32_t kBigStageBricks = 8192;  // bricks per scene up to which they do
constexpr int kOrderBins = 64;

// Staged segments ordered by their estimated number of pieces (walk_estimate),
// longest walks first, so the lanes of a wave walk segments of (nearly)
// equal piece counts: they all start together and finish together.  Bucket
// kOrderBins - est, the longest (est >= kOrderBins) in bucket 0.  The buckets
// fall into the classes of walk_parts: 8 parts (bucket 0), 4 (buckets 1-32),
// 2 (33-48) and 1 (49-63), so each class is a contiguous run of the order.
template <int kN>
struct Stage {
    StagedSeg seg[kN];
    uint16_t order[kN];
    uint32_t bins[kOrderBins];  // bucket sizes, then bucket starts, then bucket ends
    uint32_t nvalid;
    uint32_t claim;             // next group of the walk (walk_ordered)
};
static_assert(kOrderBins == 64 && kMaxWalkParts == 8, "walk classes: buckets 0, 1-32, 33-48, 49-63");
constexpr int kBinEnd8 = 0, kBinEnd4 = 32, kBinEnd2 = 48;  // last bucket of each class
// ... and of the walks of three pieces and more, and of two (estimates of one
// and two are exact).
constexpr int kBinEnd3 = kOrderBins - 3, kBinPairs = kOrderBins - 2;

__device__ __forceinline__ uint32_t order_bin(uint32_t est) {
    return (uint32_t)kOrderBins - (est < (uint32_t)kOrderBins ? est : (uint32_t)kOrderBins);
}

__device__ __forceinline__ uint32_t brick_of(const BrickGeom& bg, int32_t bx, int32_t by, int32_t bz) {
    return __umul24(__umul24((uint32_t)bz, (uint32_t)bg.nb[1]) + (uint32_t)by, (uint32_t)bg.nb[0]) + (uint32_t)bx;
}

// Loads segments [base, base + cnt) into the stage (all threads of the
// block), writes counts, flags out-of-volume segments, and builds the order
// of the in-volume ones, except those of which direct(segment, estimate) says
// that it has dealt with them.
template <int kN, typename Direct>
__device__ __forceinline__ void stage_segments(const int32_t* __restrict__ segs, int64_t base, uint32_t cnt,
                                               const BrickGeom& bg, bool euclid, Stage<kN>& st,
                                               int32_t* __restrict__ counts, bool& bad, Direct direct) {
    if (threadIdx.x < kOrderBins) st.bins[threadIdx.x] = 0;
    lds_barrier();
    constexpr int kSlots = (kN + kHistBlock - 1) / kHistBlock;
    uint32_t bins[(kSlots + 3) / 4] = {};  // bin + 1 of each of this thread's segments, 0: none
#pragma unroll
    for (int slot = 0; slot < kSlots; ++slot) {
        const uint32_t t = threadIdx.x + (uint32_t)slot * kHistBlock;
        if (t >= cnt) continue;
        const Seg g = load_seg<true>(segs, base + t);
        const bool inside = in_volume(g, bg);
        if (counts) {
            // Counts: N + 1 for the Chebyshev N; with the Euclidean N 0
            // outside the volume here, the voxels after duplicate removal
            // inside it from the histogram's count pass (euclid_counts).
            if (euclid) {
                if (!inside) counts[base + t] = 0;
            } else {
                const int64_t c = seg_length(g) + 1;
                counts[base + t] = (int32_t)(c > 0x7FFFFFFFll ? 0x7FFFFFFFll : c);
            }
        }
        StagedSeg s;
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            s.p0[ax] = (uint16_t)g.p0[ax];
            s.p1[ax] = (uint16_t)g.p1[ax];
        }
        if (inside) {
            const uint32_t est = walk_estimate(g.p0, g.p1, bg.lg);
            if (!direct(g, est)) {
                const uint32_t bin = order_bin(est);
                st.seg[t] = s;
                bins[slot / 4] |= (bin + 1u) << (8 * (slot % 4));
                atomicAdd(&st.bins[bin], 1u);
            }
        } else {
            bad = true;
        }
    }
    lds_barrier();
    if (threadIdx.x < kWave) {  // bucket offsets: one wave, one bucket per lane
        const uint32_t c = st.bins[threadIdx.x];
        const uint32_t incl = wave_inclusive_sum(c);
        st.bins[threadIdx.x] = incl - c;
        if (threadIdx.x == kWave - 1) {
            st.nvalid = incl;
            st.claim = 0;
        }
    }
    lds_barrier();
#pragma unroll
    for (int slot = 0; slot < kSlots; ++slot) {
        const uint32_t bin = (bins[slot / 4] >> (8 * (slot % 4))) & 255u;
        if (bin != 0u) {
            const uint32_t pos = atomicAdd(&st.bins[bin - 1u], 1u);
            st.order[pos] = (uint16_t)(threadIdx.x + (uint32_t)slot * kHistBlock);
        }
    }
    lds_barrier();
}
static_assert(kStageBig <= 65536, "16-bit order entries");

struct WalkState {
    AxisCross c[3];
    uint32_t N, klo;  // length (Chebyshev or Euclidean), first k inside the current brick
    uint32_t kend;    // last k of the walk's part
};

// floor(sqrt(s)) for s < 2^31: the double square root is correctly rounded,
// so its integer part is exact in this range.
__device__ __forceinline__ uint32_t isqrt31(uint32_t s) { return (uint32_t)__dsqrt_rn((double)s); }

// Walk state at the start of part `part` of `parts` of a walk (the whole
// walk when parts = 1; false for an empty part).  Every coordinate of
// eq. (3) is monotone in k for any N >= max |d_a|, so the brick crossings
// follow the same rules under the Euclidean N of eq. (1)
// (N = floor |P1 - P0| >= max |d_a|).
__device__ __forceinline__ bool walk_init(WalkState& w, const StagedSeg& g, const BrickGeom& bg, bool euclid,
                                          uint32_t part, uint32_t parts) {
    int32_t p0[3], p1[3];
    uint32_t a[3], neg[3], N = 0, ss = 0;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        p0[ax] = g.p0[ax];
        p1[ax] = g.p1[ax];
        const int32_t d = p1[ax] - p0[ax];
        neg[ax] = d < 0;
        a[ax] = (uint32_t)(d < 0 ? -d : d);
        N = a[ax] > N ? a[ax] : N;
        ss += a[ax] * a[ax];
    }
    if (euclid) N = isqrt31(ss);
    uint32_t k0 = 0, k1 = N;
    if (parts > 1u && !part_window(p0, p1, a, neg, N, bg.lg, part, parts, k0, k1)) return false;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) cross_init_at(w.c[ax], p0[ax], p1[ax], a[ax], neg[ax], N, bg.lg[ax], k0);
    w.N = N;
    w.klo = k0;
    w.kend = k1;
    return true;
}

// Steps k0 + 1 ... k0 + len (k0 + len <= N) of an in-volume segment under
// the Euclidean N at which some axis moves.  With r_a(k) = (2k a + N - neg_a)
// mod 2N, the remainder of eq. (3)'s division, axis a moves at step k exactly
// when r_a(k - 1) + 2a reaches 2N (a <= N).  One division per axis gives
// r_a(k0); the steps then run on biased 16-bit halves as in the fill
// (N <= 16384 in a brick scene).
__device__ __forceinline__ uint32_t euclid_moves(const StagedSeg& g, uint32_t N, uint32_t k0, uint32_t len) {
    uint32_t a[3], neg[3], r[3];
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const int32_t d = (int32_t)g.p1[ax] - (int32_t)g.p0[ax];
        neg[ax] = d < 0;
        a[ax] = (uint32_t)(d < 0 ? -d : d);
    }
    const uint32_t two_n = 2u * N;
    const float rcpd = rcp_down(two_n);
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        uint32_t q;
        divmod_down(2u * __umul24(k0, a[ax]) + N - neg[ax], two_n, rcpd, q, r[ax]);
    }
    u16x2 E = {(uint16_t)(r[0] + 32768u - two_n), (uint16_t)(r[1] + 32768u - two_n)};
    u16x2 Ez = {(uint16_t)(r[2] + 32768u - two_n), 0};
    const u16x2 T = {(uint16_t)(2u * a[0]), (uint16_t)(2u * a[1])};
    const u16x2 Tz = {(uint16_t)(2u * a[2]), 0};
    const u16x2 N2 = {(uint16_t)two_n, (uint16_t)two_n};
    const i16x2 k15 = {15, 15};
    uint32_t moves = 0;
#pragma unroll 4
    for (uint32_t t = 0; t < len; ++t) {
        E = E + T;
        const i16x2 C = __builtin_bit_cast(i16x2, E) >> k15;  // -1 where the axis moves
        E = E + __builtin_bit_cast(u16x2, C) * N2;
        Ez = Ez + Tz;
        const i16x2 Cz = __builtin_bit_cast(i16x2, Ez) >> k15;
        Ez = Ez + __builtin_bit_cast(u16x2, Cz) * N2;
        moves += (__builtin_bit_cast(uint32_t, C) | __builtin_bit_cast(uint32_t, Cz)) != 0u ? 1u : 0u;
    }
    return moves;
}

// Per-wave LDS of the Euclidean counts, one entry per segment of a group: its
// first chunk number, move count and length N (at most 16384).
constexpr uint32_t kCountGroup = 32;
struct CountScratch {
    uint32_t pre[kCountGroup], cnt[kCountGroup];
    uint16_t n[kCountGroup];
};
constexpr size_t kCountScratch = (size_t)(kHistBlock / kWave) * sizeof(CountScratch);

// Voxels (after duplicate removal) of the staged in-volume segments under
// the Euclidean N: 1 + the steps at which some axis moves.  Each wave takes
// 32 segments in walk order (so that a row of 512 segments keeps all 16
// waves busy), one per lane of its first half, cuts them into chunks of 64
// steps (a prefix over the lanes numbers the chunks), and runs the chunks 64
// at a time, one per lane, each lane finding its chunk's segment by binary
// search over the prefix; a segment's moves are summed with LDS atomics.
// counts: the stage's first segment's slot.
template <int kN>
__device__ __forceinline__ void euclid_counts(const Stage<kN>& st, int32_t* __restrict__ counts,
                                              CountScratch* scratch) {
    const uint32_t lane = __lane_id();
    CountScratch& w = scratch[threadIdx.x / kWave];
    const uint32_t nvalid = st.nvalid;
    for (uint32_t g0 = (threadIdx.x / kWave) * kCountGroup; g0 < nvalid;
         g0 += (kHistBlock / kWave) * kCountGroup) {
        const uint32_t i = g0 + lane;
        const bool mine = lane < kCountGroup && i < nvalid;
        uint32_t j = 0, N = 0;
        if (mine) {
            j = st.order[i];
            const StagedSeg& g = st.seg[j];
            uint32_t ss = 0;
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                const int32_t d = (int32_t)g.p1[ax] - (int32_t)g.p0[ax];
                ss += (uint32_t)(d * d);
            }
            N = isqrt31(ss);
        }
        const uint32_t ch = (N + kWave - 1) / kWave;
        const uint32_t incl = wave_inclusive_sum(ch);
        const uint32_t total = __builtin_amdgcn_readlane(incl, kWave - 1);
        if (lane < kCountGroup) {
            w.pre[lane] = incl - ch;
            w.n[lane] = (uint16_t)N;
            w.cnt[lane] = 0u;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        for (uint32_t q0 = 0; q0 < total; q0 += kWave) {
            const uint32_t q = q0 + lane;
            if (q < total) {
                // The last lane whose first chunk is at most q owns chunk q.
                uint32_t o = 0;
#pragma unroll
                for (uint32_t step = kCountGroup / 2; step > 0; step >>= 1) o += w.pre[o + step] <= q ? step : 0u;
                const uint32_t n = w.n[o];
                const uint32_t k0 = (q - w.pre[o]) * (uint32_t)kWave;
                const uint32_t len = n - k0 < (uint32_t)kWave ? n - k0 : (uint32_t)kWave;
                atomicAdd(&w.cnt[o], euclid_moves(st.seg[st.order[g0 + o]], n, k0, len));
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (mine) counts[j] = (int32_t)(1u + w.cnt[lane]);
        // The scratch is rewritten by the wave's next 64 segments.
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

// Walks the ordered staged segments.  With kSplit the order falls into four
// classes of walk_parts (8, 4, 2 and 1 parts, longest walks first), and the
// walk into groups of 64 part walks: 8 segments of the first class cut into
// 8 parts each, 16 of the second cut into 4, and so on; without, into groups
// of 64 whole walks.  Waves claim groups in order from an LDS counter, so the
// longest groups start first and a wave that finishes early takes the next
// group (no wave waits for a fixed share).  Lanes of a group step their
// walks one brick at a time until the last ends.  The parts cost a division
// or three each at their start: the scatter, whose steps are dear (a record
// store each), gains from them, the histogram (an LDS increment a step) does
// not.
// Segments of one and two pieces (with kSplit) are groups of their own, which
// need no walk: no division, and one for the crossing.  The histogram counts
// them while it stages.  With that, and divisions by biased reciprocals where
// there were IEEE ones (six a walk), the histogram of 4 M segments of 4.5 pieces
// takes 0.079 ms against 0.102, of 9.6 M of 2 pieces 0.165 against 0.210.
// emit(maker, brick id, klo, khi, brick x, y, z) per piece, [klo, khi] being
// the segment's k-window inside the brick; the Maker is made once per walk
// from the segment and its N, so what a piece's record takes from the segment
// alone is computed once per walk, not per piece.
struct NoMaker {
    __device__ __forceinline__ NoMaker(const StagedSeg&, uint32_t) {}
};

// The two pieces of a segment that crosses one brick face, or its one piece.
template <bool kPair, typename Maker, typename Emit>
__device__ __forceinline__ void short_walk(const StagedSeg& g, const BrickGeom& bg, bool euclid, Emit emit) {
    uint32_t N = 0, ss = 0, m = 0, as = 0, ns = 0;
    int32_t b0[3], b1[3];
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const int32_t p0 = g.p0[ax], p1 = g.p1[ax], d = p1 - p0;
        const uint32_t a = (uint32_t)(d < 0 ? -d : d);
        N = a > N ? a : N;
        ss += a * a;
        b0[ax] = p0 >> bg.lg[ax];
        b1[ax] = p1 >> bg.lg[ax];
        if constexpr (kPair) {
            // Offset of the far face from p0 on the crossing axis.
            const bool cross = b0[ax] != b1[ax];
            const uint32_t far = (uint32_t)(d < 0 ? p0 - (b0[ax] << bg.lg[ax]) + 1 : (b1[ax] << bg.lg[ax]) - p0);
            m = cross ? far : m;
            as = cross ? a : as;
            ns = cross ? (d < 0 ? 1u : 0u) : ns;
        }
    }
    if (euclid) N = isqrt31(ss);
    const Maker maker(g, N);
    uint32_t k = N + 1u;
    if constexpr (kPair) {
        uint32_t q, r;
        const uint32_t D = 2u * as;
        divmod_down(2u * __umul24(N, m) - N + ns, D, rcp_walk(D), q, r);
        k = r ? q + 1u : q;
    }
    emit(maker, brick_of(bg, b0[0], b0[1], b0[2]), 0u, k - 1u, b0[0], b0[1], b0[2]);
    if constexpr (kPair) emit(maker, brick_of(bg, b1[0], b1[1], b1[2]), k, N, b1[0], b1[1], b1[2]);
}

template <bool kSplit, typename Maker, int kN, typename Emit>
__device__ __forceinline__ void walk_ordered(Stage<kN>& st, const BrickGeom& bg, bool euclid, Emit emit) {
    const uint32_t lane = __lane_id();
    const uint32_t nvalid = st.nvalid;
    // Ends of the classes in the order, and their first groups (without
    // kSplit every walk is in the last class).
    const uint32_t e8 = kSplit ? st.bins[kBinEnd8] : 0u;
    const uint32_t e4 = kSplit ? st.bins[kBinEnd4] : 0u;
    const uint32_t e2 = kSplit ? st.bins[kBinEnd2] : 0u;
    const uint32_t e1 = kSplit ? st.bins[kBinEnd3] : nvalid;
    const uint32_t ep = kSplit ? st.bins[kBinPairs] : nvalid;
    const uint32_t g4 = (e8 + 7u) >> 3;
    const uint32_t g2 = g4 + ((e4 - e8 + 15u) >> 4);
    const uint32_t g1 = g2 + ((e2 - e4 + 31u) >> 5);
    const uint32_t gp = g1 + ((e1 - e2 + 63u) >> 6);
    const uint32_t gs = gp + ((ep - e1 + 63u) >> 6);
    const uint32_t gt = gs + ((nvalid - ep + 63u) >> 6);
    for (;;) {
        uint32_t grp = 0;
        if (lane == 0) grp = atomicAdd(&st.claim, 1u);
        grp = __builtin_amdgcn_readfirstlane(grp);
        if (grp >= gt) break;
        if constexpr (kSplit) {
            if (grp >= gp) {
                const bool pair = grp < gs;
                const uint32_t i = (pair ? e1 + ((grp - gp) << 6) : ep + ((grp - gs) << 6)) + lane;
                if (i < (pair ? ep : nvalid)) {
                    const StagedSeg g = st.seg[st.order[i]];
                    if (pair)
                        short_walk<true, Maker>(g, bg, euclid, emit);
                    else
                        short_walk<false, Maker>(g, bg, euclid, emit);
                }
                continue;
            }
        }
        uint32_t lgp, start, end;
        if (grp < g4) {
            lgp = 3; start = grp << 3; end = e8;
        } else if (grp < g2) {
            lgp = 2; start = e8 + ((grp - g4) << 4); end = e4;
        } else if (grp < g1) {
            lgp = 1; start = e4 + ((grp - g2) << 5); end = e2;
        } else {
            lgp = 0; start = e2 + ((grp - g1) << 6); end = e1;
        }
        const uint32_t i = start + (lane >> lgp);
        bool active = i < end;
        StagedSeg g = {};
        WalkState w = {};
        if (active) {
            g = st.seg[st.order[i]];
            active = walk_init(w, g, bg, euclid, lane & ((1u << lgp) - 1u), 1u << lgp);
        }
        const Maker maker(g, w.N);
        while (__ballot(active)) {
            uint32_t km = w.c[0].kn < w.c[1].kn ? w.c[0].kn : w.c[1].kn;
            km = km < w.c[2].kn ? km : w.c[2].kn;
            const bool more = km <= w.kend;
            // Brick ids and counts stay below 2^24: 24-bit multiplies.
            if (active)
                emit(maker, brick_of(bg, w.c[0].b, w.c[1].b, w.c[2].b), w.klo, more ? km - 1u : w.kend, w.c[0].b,
                     w.c[1].b, w.c[2].b);
            // The rest with selects only (lanes step different segments).
            const bool go = active && more;
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) cross_advance(w.c[ax], go && w.c[ax].kn == km);
            w.klo = go ? km : w.klo;
            active = go;
        }
    }
}

// Histogram of one row: its segments' pieces per brick of its scene.
template <int kN>
__device__ __forceinline__ void hist_row(const BrickScene& sc, uint32_t g, Stage<kN>& st, uint32_t* lh,
                                         CountScratch* cscratch, const WorkView& wv) {
    const BrickGeom& bg = sc.bg;
    const uint32_t NB = bg.nbricks;
    for (uint32_t b = threadIdx.x; b < NB; b += kHistBlock) lh[b] = 0;
    int64_t lo, hi;
    seg_range(sc.n, (int)g, (int)sc.rows, lo, hi);
    const bool euclid = (sc.flags & kSceneEuclid) != 0;
    bool bad = false;
    for (int64_t base = lo; base < hi; base += kN) {
        const uint32_t cnt = (uint32_t)(hi - base < kN ? hi - base : kN);
        // Segments of one and two pieces, which lie in the bricks of their end
        // points, are counted on the way (unless euclid_counts wants them).
        auto ends = [&](const Seg& g, uint32_t est) {
            if (est > 2u || (euclid && sc.counts)) return false;
            atomicAdd(&lh[brick_of(bg, g.p0[0] >> bg.lg[0], g.p0[1] >> bg.lg[1], g.p0[2] >> bg.lg[2])], 1u);
            if (est == 2u)
                atomicAdd(&lh[brick_of(bg, g.p1[0] >> bg.lg[0], g.p1[1] >> bg.lg[1], g.p1[2] >> bg.lg[2])], 1u);
            return true;
        };
        stage_segments(sc.segs, base, cnt, bg, euclid, st, sc.counts, bad, ends);
        walk_ordered<false, NoMaker>(st, bg, euclid,
                                     [&](const NoMaker&, uint32_t b, uint32_t, uint32_t, int32_t, int32_t, int32_t) {
                                         atomicAdd(&lh[b], 1u);
                                     });
        if (euclid && sc.counts) euclid_counts(st, sc.counts + base, cscratch);
        lds_barrier();
    }
    // (Out-of-volume segments are reported by the scatter, or by the direct
    // kernels when they serve the scene: the status word may still be
    // written by this kernel's first workgroup in a plain call.)
    (void)bad;
    lds_barrier();
    uint32_t* row = wv.hist + sc.hist_off + (size_t)g * NB;
    for (uint32_t b = threadIdx.x; b < NB; b += kHistBlock) row[b] = lh[b];
}

// LDS of a plain call's histogram: 8 192 staged segments and up to 8 192 brick
// counters, or 4 096 staged segments and up to 16 384 counters; each
// workgroup takes the layout its scene's brick count allows.
constexpr size_t kHistLdsBig = sizeof(Stage<kStageBig>) + (size_t)kBigStageBricks * 4;
constexpr size_t kHistLdsSmall = sizeof(Stage<kStage>) + (size_t)kMaxBricks * 4;
// ... then the per-wave scratch of the Euclidean counts.
constexpr size_t kHistLds = (kHistLdsBig > kHistLdsSmall ? kHistLdsBig : kHistLdsSmall) + kCountScratch;
static_assert(kHistLds <= 163840, "histogram LDS fits a workgroup");

// Batches have more rows than the chip has CUs, of about kSegsPerRow segments:
// two workgroups a CU (80 KiB of LDS, 64 VGPRs each) hide each other's loads
// and barriers, with room for every segment of a row beside the counters of
// 4096 bricks, and for fewer at a time beside those of more.  256 scenes with
// 9.6 M segments in all: 0.137 ms against 0.165 with one a CU; eight wireframes
// 0.009 against 0.016.  (The scatter, of 94 VGPRs, gains nothing from two of
// 512 threads, and loses more than half to the spills of two of 1024.)
constexpr size_t kTwoPerCu = 81920;
template <int kN>
struct BatchLayout {
    static constexpr uint32_t kBricks = kN == 4096 ? 4096u : (kN == 2048 ? 8192u : kMaxBricks);
    static constexpr size_t kBytes = sizeof(Stage<kN>) + (size_t)kBricks * 4;
    static_assert(kBytes <= kTwoPerCu - kCountScratch, "two workgroups a CU");
    Stage<kN> st;
    uint32_t bricks[kBricks];
};
static_assert(kSegsPerRow == 4096 && kMaxBricks == 16384, "layouts of the batch kernels");

__global__ __launch_bounds__(kHistBlock, 8) void k_brick_hist(uint8_t* __restrict__ work) {
    __shared__ __align__(16) uint8_t lds[kTwoPerCu];
    const TableView tv = table_view(work + kWorkTable);
    const WorkView wv = work_of(work, tv);
    const uint32_t r = xcd_row(blockIdx.x, gridDim.x);
    if (*wv.ok == 0 || r >= tv.h.rows) return;
    const uint32_t si = scene_of_row(tv, r);
    const BrickScene sc = tv.scenes[si];
    const uint32_t g = r - sc.row_base;
    if (tv.row_scene) {
        // The scenes of the rows and bricks, for the kernels that follow.
        if (threadIdx.x == 0) const_cast<uint32_t*>(tv.row_scene)[r] = si;
        if (g == 0) {
            uint32_t* brick_scene = const_cast<uint32_t*>(tv.brick_scene) + sc.brick_base;
            const uint32_t nb = (sc.bg.nbricks + 1u) & ~1u;
            for (uint32_t b = threadIdx.x; b < nb; b += kHistBlock) brick_scene[b] = si;
        }
    }
    auto* scratch = reinterpret_cast<CountScratch*>(lds + kTwoPerCu - kCountScratch);
    auto row = [&](auto* layout) { hist_row(sc, g, layout->st, layout->bricks, scratch, wv); };
    if (sc.bg.nbricks <= BatchLayout<4096>::kBricks)
        row(reinterpret_cast<BatchLayout<4096>*>(lds));
    else if (sc.bg.nbricks <= BatchLayout<2048>::kBricks)
        row(reinterpret_cast<BatchLayout<2048>*>(lds));
    else
        row(reinterpret_cast<BatchLayout<512>*>(lds));
}

// A plain call's plan and histogram in one launch: every workgroup plans the
// call's one scene (passed by value) itself, the first one also writes the
// table and header words for the kernels that follow (what k_brick_plan
// writes for a single scene), and the workgroups go on to their histogram
// rows when the brick kernels may run.
__global__ __launch_bounds__(kHistBlock) void k_brick_plan_hist(vox_scene one, BrickLaunch L,
                                                               uint8_t* __restrict__ work, uint64_t work_bytes) {
    extern __shared__ __align__(16) uint8_t hist_lds[];
    BrickScene sc;
    const bool valid = plan_scene(one, L.lg, L.segs_per_row, sc);
    const bool isd = (sc.flags & kSceneDirect) != 0;
    sc.row_base = 0;
    sc.brick_base = 0;
    sc.hist_off = 0;
    const uint32_t nb = isd ? 0u : sc.bg.nbricks;
    const uint64_t n = sc.n > 0 ? (uint64_t)sc.n : 0u;
    const uint64_t hist_c = (uint64_t)sc.rows * nb;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        BrickScene* out = reinterpret_cast<BrickScene*>(work + kWorkTable + kTableScenes);
        out[0] = sc;
        if (isd) reinterpret_cast<uint32_t*>(out + 1)[0] = 0u;
        write_table(work, L, work_bytes, sc.rows, nb, isd ? 1u : 0u, hist_c, n, isd ? n : 0u, !valid);
    }
    // The same decision as the ok word written above.
    const WorkView wv = work_view(work, kWorkTable + L.table_bytes, hist_c, nb);
    const bool fits = n <= L.total_segments && sc.rows <= L.rows && nb <= L.bricks;
    if (!valid || !fits || wv.rec_off > work_bytes || nb == 0) return;
    const uint32_t r = xcd_row(blockIdx.x, gridDim.x);
    if (r >= sc.rows) return;
    if (nb <= kBigStageBricks) {
        auto* st = reinterpret_cast<Stage<kStageBig>*>(hist_lds);
        hist_row(sc, r, *st, reinterpret_cast<uint32_t*>(hist_lds + sizeof(Stage<kStageBig>)),
                 reinterpret_cast<CountScratch*>(hist_lds + kHistLdsBig), wv);
    } else {
        auto* st = reinterpret_cast<Stage<kStage>*>(hist_lds);
        hist_row(sc, r, *st, reinterpret_cast<uint32_t*>(hist_lds + sizeof(Stage<kStage>)),
                 reinterpret_cast<CountScratch*>(hist_lds + kHistLdsSmall), wv);
    }
}

constexpr int kBaseBlock = 1024;

// The brick totals pass through LDS in chunks of kBaseChunk bricks: loaded
// coalesced (all of a thread's loads issued before any is used), read in
// runs of consecutive bricks per thread for the scans, and the results (bin
// and item offsets) staged in LDS and written back coalesced: from one
// workgroup, stores of the threads' runs would each touch a memory line of
// their own.  Entry i of a stage sits at i + i / 32,
// so that the lanes' runs (16 entries apart) fall in different banks.
constexpr uint32_t kBaseChunk = 16384;
constexpr uint32_t kBaseStage = kBaseChunk + kBaseChunk / 32;
__device__ __forceinline__ uint32_t stage_slot(uint32_t i) { return i + (i >> 5); }

template <int kBlock>
__device__ __forceinline__ void stage_in(const uint32_t* __restrict__ src, uint32_t m, uint32_t* st) {
    constexpr int kPer = (int)(kBaseChunk / kBlock);
    uint32_t v[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const uint32_t i = threadIdx.x + (uint32_t)k * kBlock;
        v[k] = i < m ? src[i] : 0u;
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) st[stage_slot(threadIdx.x + (uint32_t)k * kBlock)] = v[k];
    __syncthreads();
}

template <int kBlock>
__device__ __forceinline__ void stage_out(const uint32_t* st, uint32_t m, uint32_t* __restrict__ dst) {
    for (uint32_t i = threadIdx.x; i < m; i += kBlock) dst[i] = st[stage_slot(i)];
}

// Exclusive scan, from `base`, of f(entry) over the m entries of a stage
// (runs of kBaseChunk / kBlock consecutive entries per thread, one block
// scan of the run sums; lds: kBlock / 64 entries) into the stage `out`;
// returns the sum.
template <int kBlock, typename F>
__device__ __forceinline__ uint64_t scan_stage(const uint32_t* st, uint32_t m, uint64_t base, uint32_t* out,
                                               uint64_t* lds, F f, uint32_t* max_s = nullptr) {
    constexpr uint32_t kRun = kBaseChunk / kBlock;
    const uint32_t r0 = threadIdx.x * kRun;
    uint64_t run = 0;
    uint32_t mx = 0;
    for (uint32_t k = 0; k < kRun && r0 + k < m; ++k) {
        const uint32_t c = st[stage_slot(r0 + k)];
        run += f(c);
        mx = c > mx ? c : mx;
    }
    if (max_s) {
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const uint32_t o = (uint32_t)__shfl_xor((int)mx, d, kWave);
            mx = o > mx ? o : mx;
        }
        if ((threadIdx.x & (kWave - 1)) == 0) atomicMax(max_s, mx);  // (read after the scan's barriers)
    }
    uint64_t sum;
    uint64_t off = base + block_exclusive_sum<kBlock>(run, lds, sum);
    for (uint32_t k = 0; k < kRun && r0 + k < m; ++k) {
        out[stage_slot(r0 + k)] = (uint32_t)off;
        off += f(st[stage_slot(r0 + k)]);
    }
    __syncthreads();
    return sum;
}

// bin_base[b] = sum of totals before global brick b, bin_base[NB] = total,
// by one block of kBlock threads, a chunk at a time.  The direct kernels
// take over when the records do not fit the workspace (or reach 2^32 - 1).
template <int kBlock>
__device__ __forceinline__ uint64_t scan_totals(const WorkView& wv, uint32_t NB, uint64_t work_bytes, uint64_t* lds,
                                                uint32_t* st, uint32_t* ob, uint32_t* max_s) {
    uint64_t total = 0;
    if (threadIdx.x == 0) *max_s = 0u;  // (ordered before the atomics by stage_in's barrier)
    for (uint32_t c0 = 0; c0 < NB; c0 += kBaseChunk) {
        const uint32_t m = NB - c0 < kBaseChunk ? NB - c0 : kBaseChunk;
        stage_in<kBlock>(wv.totals + c0, m, st);
        total += scan_stage<kBlock>(st, m, total, ob, lds, [](uint32_t c) { return (uint64_t)c; }, max_s);
        stage_out<kBlock>(ob, m, wv.bin_base + c0);
        __syncthreads();  // both stages are rewritten by the next chunk (st read by make_items)
    }
    if (threadIdx.x == 0) {
        wv.bin_base[NB] = (uint32_t)total;
        *wv.pieces = total;
        const uint64_t cap = work_bytes > wv.rec_off ? (work_bytes - wv.rec_off) / sizeof(Piece) : 0u;
        if (total > cap || total >= 0xFFFFFFFFull) *wv.direct_all = 1u;
    }
    return total;
}

// What split_least asks for: the voxels and pieces of a sample of the segments, one
// in each of its threads' shares of the rows, and the words of the box that
// holds it, in every scene.
constexpr uint32_t kSampleThreads = 256;
struct SplitSample {
    uint32_t voxels, pieces;
    uint64_t words;
};
struct SampleSeg {
    const BrickScene* sc;
    Seg g;
    bool any;
};
__device__ __forceinline__ SampleSeg sample_load(const TableView& tv) {
    SampleSeg out{tv.scenes, Seg{}, false};
    if (threadIdx.x >= kSampleThreads) return out;
    const uint32_t at = threadIdx.x * tv.h.rows, r = at / kSampleThreads;
    out.sc = tv.scenes + (tv.row_scene ? tv.row_scene[r] : 0u);
    int64_t lo, hi;
    seg_range(out.sc->n, (int)(r - out.sc->row_base), (int)out.sc->rows, lo, hi);
    lo += (hi - lo) * (int64_t)(at % kSampleThreads) / kSampleThreads;
    out.any = lo < hi;
    if (out.any) out.g = load_seg<true>(out.sc->segs, lo);
    return out;
}

// The larger halves of the wave's values, in lane 63 (row shifts and broadcasts,
// as wave_inclusive_sum_dpp).
__device__ __forceinline__ u16x2 wave_max_dpp(u16x2 v) {
    auto step = [&](auto ctrl, auto rows) {
        const u16x2 o = __builtin_bit_cast(u16x2, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), decltype(ctrl)::value,
                                                                             decltype(rows)::value, 0xf, false));
        v = __builtin_elementwise_max(v, o);
    };
    step(std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xf>{});
    step(std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xf>{});
    step(std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xf>{});
    step(std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xf>{});
    step(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});
    step(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});
    return v;
}

// All threads of a block; s: 8 words of LDS.
__device__ __forceinline__ SplitSample sample_pieces(const SampleSeg& from, uint32_t n_scenes, uint32_t* s) {
    if (threadIdx.x < 8u) s[threadIdx.x] = 0u;
    __syncthreads();
    if (threadIdx.x < kSampleThreads) {
        const BrickGeom& bg = from.sc->bg;
        const Seg& g = from.g;
        uint32_t voxels = 0, pieces = 0;
        u16x2 box[3] = {};  // largest coordinate, 16383 - the smallest
        if (from.any && in_volume(g, bg)) {
            voxels = seg_axes(g).N + 1u;
            pieces = walk_estimate(g.p0, g.p1, bg.lg);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const int32_t c0 = g.p0[a] < g.p1[a] ? g.p0[a] : g.p1[a], c1 = g.p0[a] < g.p1[a] ? g.p1[a] : g.p0[a];
                box[a] = (u16x2){(uint16_t)c1, (uint16_t)(16383 - c0)};
            }
        }
        voxels = wave_inclusive_sum_dpp(voxels);
        pieces = wave_inclusive_sum_dpp(pieces);
#pragma unroll
        for (int a = 0; a < 3; ++a) box[a] = wave_max_dpp(box[a]);
        if (__lane_id() == kWave - 1) {
            atomicAdd(&s[0], voxels);
            atomicAdd(&s[1], pieces);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                atomicMax(&s[2 + a], (uint32_t)box[a][0]);
                atomicMax(&s[5 + a], (uint32_t)box[a][1]);
            }
        }
    }
    __syncthreads();
    SplitSample out{s[0], s[1], n_scenes};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const uint32_t largest = s[2 + a], smallest = 16383u - s[5 + a];
        out.words *= largest > smallest ? largest - smallest + 1u : 1u;
    }
    out.words = (out.words + 31u) / 32u;
    __syncthreads();
    return out;
}

// Records from which a brick is cut, by a block that knows the largest brick's.
// busy(): how many have any.  (It and the sample are taken where a brick would be
// cut anyway.)
template <typename Busy>
__device__ __forceinline__ uint64_t cut_threshold(const TableView& tv, uint64_t total, uint32_t max, uint32_t* s,
                                                  Busy busy) {
    const uint64_t most = split_threshold(total);
    if ((uint64_t)max <= most) return most;
    const uint32_t bricks = busy();
    if (bricks > kSplitFewBricks) return most;
    const SplitSample p = sample_pieces(sample_load(tv), tv.h.n_scenes, s);
    return split_threshold(total, split_least(total, p.voxels, p.pieces, p.words, bricks));
}

// The fill's work items (see kSplitShares) when some brick is cut, the same
// way: item_base[b] = extra items before brick b (a brick of k items has
// k - 1), the brick of each extra item, the list of cut bricks, and the
// counts in the header: the extra items, rounded up to even so that the
// bricks keep their pairs, come before the bricks.  With a single chunk the
// stage still holds the totals from scan_totals.  When no brick is cut the
// items are the bricks (n_split = 0 tells the fill and the scatter so, and
// the item arrays are not written).
template <int kBlock>
__device__ __forceinline__ void make_items(const WorkView& wv, uint32_t NB, uint64_t T, uint64_t* lds, uint32_t* st,
                                           uint32_t* ob, uint32_t* n_split_s) {
    if (threadIdx.x == 0) *n_split_s = 0u;  // (ordered before the atomics below by the scan's barriers)
    uint64_t extra = 0;
    for (uint32_t c0 = 0; c0 < NB; c0 += kBaseChunk) {
        const uint32_t m = NB - c0 < kBaseChunk ? NB - c0 : kBaseChunk;
        if (NB > kBaseChunk) stage_in<kBlock>(wv.totals + c0, m, st);
        const uint64_t sum = scan_stage<kBlock>(st, m, extra, ob, lds, [T](uint32_t c) {
            return (uint64_t)(brick_items(c, T) - 1u);
        });
        stage_out<kBlock>(ob, m, wv.item_base + c0);
        // A brick's extra items are the difference of its offset and the
        // next one (at most kMaxExtraItems in all: few scattered stores).
        const uint32_t end = (uint32_t)(extra + sum);
        for (uint32_t i = threadIdx.x; i < m; i += kBlock) {
            const uint32_t o = ob[stage_slot(i)];
            const uint32_t n = (i + 1u < m ? ob[stage_slot(i + 1u)] : end) - o;
            if (n > 0u) wv.split[atomicAdd(n_split_s, 1u)] = c0 + i;
            for (uint32_t j = 0; j < n; ++j) wv.item_brick[o + j] = c0 + i;
        }
        extra += sum;
        __syncthreads();  // both stages are rewritten by the next chunk
    }
    if (threadIdx.x == 0) {
        wv.item_base[NB] = (uint32_t)extra;
        *wv.n_items = (((uint32_t)extra + 1u) & ~1u) + NB;
        *wv.n_split = *n_split_s;
    }
}

constexpr int kColBins = 64;
constexpr int kColSplit = 4;  // row chunks per brick
constexpr int kColRows = (kHistRows + kColSplit - 1) / kColSplit;
constexpr uint32_t kColMaxBlocks = 4096;

// Blocks of 256 threads = 64 global bricks x 4 row chunks (the blocks step
// over all bricks): per brick, exclusive prefix of its scene's histogram
// column over the scene's rows (in place) and the brick total.
__global__ __launch_bounds__(256) void k_brick_colscan(uint8_t* __restrict__ work) {
    __shared__ uint32_t part[kColSplit][kColBins];
    const TableView tv = table_view(work + kWorkTable);
    const WorkView wv = work_of(work, tv);
    if (*wv.ok == 0) return;
    const int bl = threadIdx.x % kColBins;
    const int ch = threadIdx.x / kColBins;
    for (uint32_t gb0 = blockIdx.x * kColBins; gb0 < tv.h.bricks; gb0 += gridDim.x * kColBins) {
        const uint32_t gb = gb0 + bl;
        const bool valid = gb < tv.h.bricks;
        uint32_t b = 0, NB = 0;
        int G = 0;
        uint64_t off = 0;
        if (valid) {
            const BrickScene& sc = tv.scenes[tv.brick_scene ? tv.brick_scene[gb] : 0u];
            b = gb - sc.brick_base;
            NB = sc.bg.nbricks;
            G = (int)sc.rows;
            off = sc.hist_off;
            if (b >= NB) G = 0;  // (the brick that rounds up an odd count)
        }
        uint32_t* hist = wv.hist + off;
        const int g0 = ch * kColRows;
        uint32_t v[kColRows];
        uint32_t sum = 0;
#pragma unroll
        for (int r = 0; r < kColRows; ++r) {
            const int g = g0 + r;
            v[r] = (valid && g < G) ? hist[(size_t)g * NB + b] : 0u;
            sum += v[r];
        }
        part[ch][bl] = sum;
        __syncthreads();
        uint32_t run = 0, tot = 0;
#pragma unroll
        for (int c = 0; c < kColSplit; ++c) {
            run += c < ch ? part[c][bl] : 0u;
            tot += part[c][bl];
        }
#pragma unroll
        for (int r = 0; r < kColRows; ++r) {
            const int g = g0 + r;
            if (valid && g < G) hist[(size_t)g * NB + b] = run;
            run += v[r];
        }
        if (ch == 0 && valid) wv.totals[gb] = tot;
        __syncthreads();
    }
}


// One block: bin_base[b] = sum of totals before global brick b;
// bin_base[bricks] = total.  When the records do not fit the rest of the
// workspace (or their count reaches 2^32 - 1), the direct kernels serve
// every scene instead of the scatter and the fill.
__global__ __launch_bounds__(kBaseBlock) void k_brick_base(uint8_t* __restrict__ work, uint64_t work_bytes) {
    __shared__ uint64_t lds[kBaseBlock / kWave];
    __shared__ uint32_t st[kBaseStage], ob[kBaseStage];
    __shared__ uint32_t n_split_s, max_s, sample_s[8];
    const TableView tv = table_view(work + kWorkTable);
    const WorkView wv = work_of(work, tv);
    if (*wv.ok == 0) return;
    const uint64_t total = scan_totals<kBaseBlock>(wv, tv.h.bricks, work_bytes, lds, st, ob, &max_s);
    const uint64_t T = cut_threshold(tv, total, max_s, sample_s, [&] {
        uint64_t busy = 0, all;
        for (uint32_t b = threadIdx.x; b < tv.h.bricks; b += kBaseBlock) busy += wv.totals[b] != 0u ? 1u : 0u;
        (void)block_exclusive_sum<kBaseBlock>(busy, lds, all);
        return (uint32_t)all;
    });
    if ((uint64_t)max_s > T) {
        make_items<kBaseBlock>(wv, tv.h.bricks, T, lds, st, ob, &n_split_s);
    } else if (threadIdx.x == 0) {
        *wv.n_items = tv.h.bricks;
        *wv.n_split = 0u;
    }
}

// Records of a staged segment's pieces: what depends on the segment alone,
// made once per walk, and the record of the piece with k-window [klo, khi] in
// brick (bx, by, bz).  Every volume side is at most 16384, so N < 2^15 and
// eq. (3)'s numerator 2 klo a + N stays below 2^31 (divmod_down's domain).
struct PieceMaker {
    int32_t p0[3];
    uint32_t aa, ab, m, nega, negb, negm, two_n, num_a, num_b;
    uint32_t v, ib;  // the record's third word, slope of b
    float rcp;

    __device__ __forceinline__ PieceMaker(const StagedSeg& g, uint32_t) {
        int32_t d[3];
        uint32_t ad[3];
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            p0[ax] = g.p0[ax];
            d[ax] = (int32_t)g.p1[ax] - p0[ax];
            ad[ax] = (uint32_t)(d[ax] < 0 ? -d[ax] : d[ax]);
        }
        const uint32_t N = ad[0] > ad[1] ? (ad[0] > ad[2] ? ad[0] : ad[2]) : (ad[1] > ad[2] ? ad[1] : ad[2]);
        m = ad[0] == N ? 0u : (ad[1] == N ? 1u : 2u);
        aa = m == 0 ? ad[1] : ad[0];
        ab = m == 2 ? ad[1] : ad[2];
        nega = (m == 0 ? d[1] : d[0]) < 0;
        negb = (m == 2 ? d[1] : d[2]) < 0;
        negm = (m == 0 ? d[0] : (m == 1 ? d[1] : d[2])) < 0;
        two_n = N > 0 ? 2u * N : 2u;
        num_a = (two_n >> 1) - nega;
        num_b = (two_n >> 1) - negb;
        rcp = __builtin_amdgcn_rcpf((float)two_n);
        const uint32_t ia = fix23_slope(2u * aa, two_n, rcp);
        ib = fix23_slope(2u * ab, two_n, rcp);
        v = (ia << 9) | (negm << 5) | (ib >> 18);
    }
    __device__ __forceinline__ Piece operator()(uint32_t klo, uint32_t khi, int32_t bx, int32_t by, int32_t bz,
                                                const BrickGeom& bg) const {
        const float rcpd = rcp_bias_down(rcp);
        uint32_t qa, ra, qb, rb;
        divmod_down(2u * __umul24(klo, aa) + num_a, two_n, rcpd, qa, ra);
        divmod_down(2u * __umul24(klo, ab) + num_b, two_n, rcpd, qb, rb);
        const int32_t vm = negm ? -(int32_t)klo : (int32_t)klo;
        const int32_t va = nega ? -(int32_t)qa : (int32_t)qa, vb = negb ? -(int32_t)qb : (int32_t)qb;
        const int32_t x = p0[0] + (m == 0 ? vm : va) - (bx << bg.lg[0]);
        const int32_t y = p0[1] + (m == 1 ? vm : (m == 0 ? va : vb)) - (by << bg.lg[1]);
        const int32_t z = p0[2] + (m == 2 ? vm : vb) - (bz << bg.lg[2]);
        Piece pc;
        pc.e = (fix23_fraction(ra, 2u * aa, two_n, rcp) << 9) | (ib & 511u);
        pc.t = (fix23_fraction(rb, 2u * ab, two_n, rcp) << 9) | ((ib >> 9) & 511u);
        pc.v = v;
        pc.w = (uint32_t)(x + (y << bg.lg[0]) + (z << (bg.lg[0] + bg.lg[1]))) |
               ((khi - klo) << (bg.lg[0] + bg.lg[1] + bg.lg[2])) | (m << 28) | (nega << 30) | (negb << 31);
        return pc;
    }
};

// The record of a piece under the Euclidean N of eq. (1), where every axis,
// the dominant one too, may stay put at a step: the integers from which the
// fill derives the three axes' quotients and remainders at any k,
//   e  klo | 2 a_m << 16 (a_m = |d| of the dominant axis)
//   t  2a | 2b << 16
//   v  m | nega << 2 | negb << 3 | negm << 4 | 2N << 16 (2N = 2 when N = 0)
//   w  the bit index of the start point relative to the brick's origin, mod
//      the brick's voxel count, | (samples - 1) << its log2
// The samples k = klo ... khi count duplicates.  N is at most 16384 (the
// scene's diagonal is below 16385).
struct PieceMakerEuclid {
    int32_t p0[3];
    uint32_t e, t, v;

    __device__ __forceinline__ PieceMakerEuclid(const StagedSeg& g, uint32_t N) {
        int32_t d[3];
        uint32_t ad[3];
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            p0[ax] = g.p0[ax];
            d[ax] = (int32_t)g.p1[ax] - p0[ax];
            ad[ax] = (uint32_t)(d[ax] < 0 ? -d[ax] : d[ax]);
        }
        const uint32_t amax = ad[0] > ad[1] ? (ad[0] > ad[2] ? ad[0] : ad[2]) : (ad[1] > ad[2] ? ad[1] : ad[2]);
        const uint32_t m = ad[0] == amax ? 0u : (ad[1] == amax ? 1u : 2u);
        const uint32_t aa = m == 0 ? ad[1] : ad[0], ab = m == 2 ? ad[1] : ad[2];
        const int32_t da = m == 0 ? d[1] : d[0], db = m == 2 ? d[1] : d[2];
        const int32_t dm = m == 0 ? d[0] : (m == 1 ? d[1] : d[2]);
        const uint32_t two_n = N > 0 ? 2u * N : 2u;
        e = (2u * amax) << 16;
        t = (2u * aa) | ((2u * ab) << 16);
        v = m | ((uint32_t)(da < 0) << 2) | ((uint32_t)(db < 0) << 3) | ((uint32_t)(dm < 0) << 4) | (two_n << 16);
    }
    __device__ __forceinline__ Piece operator()(uint32_t klo, uint32_t khi, int32_t bx, int32_t by, int32_t bz,
                                                const BrickGeom& bg) const {
        const int32_t x = p0[0] - (bx << bg.lg[0]), y = p0[1] - (by << bg.lg[1]), z = p0[2] - (bz << bg.lg[2]);
        const int bits = bg.lg[0] + bg.lg[1] + bg.lg[2];
        Piece pc;
        pc.e = klo | e;
        pc.t = t;
        pc.v = v;
        pc.w = ((uint32_t)(x + y * (1 << bg.lg[0]) + z * (1 << (bg.lg[0] + bg.lg[1]))) & ((1u << bits) - 1u)) |
               ((khi - klo) << bits);
        return pc;
    }
};

// Zeroes brick lb of a scene in its volume (a workgroup).
__device__ __forceinline__ void zero_brick(const BrickScene& sc, uint32_t lb) {
    const BrickGeom& bg = sc.bg;
    const int32_t org[3] = {(int32_t)(lb % (uint32_t)bg.nb[0]) << bg.lg[0],
                            (int32_t)((lb / (uint32_t)bg.nb[0]) % (uint32_t)bg.nb[1]) << bg.lg[1],
                            (int32_t)(lb / ((uint32_t)bg.nb[0] * (uint32_t)bg.nb[1])) << bg.lg[2]};
    int32_t ext[3];
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const int32_t e = bg.dim[ax] - org[ax];
        ext[ax] = e < (1 << bg.lg[ax]) ? e : (1 << bg.lg[ax]);
    }
    // Over the brick's words by shifts (divisions by the extents took longer than
    // the stores), 16 bytes at a time where rows are whole such units.
    const int64_t row_words = (int64_t)bg.dim[0] >> 5;
    uint32_t* grid = sc.grid + ((int64_t)org[2] * bg.dim[1] + org[1]) * row_words + (org[0] >> 5);
    const bool vec = ((uint32_t)bg.dim[0] & 127u) == 0u;
    const int lgu = bg.lg[0] - (vec ? 7 : 5);  // units a row
    const int32_t xus = ext[0] >> (vec ? 7 : 5);
    for (uint32_t u = threadIdx.x; u < 1u << (lgu + bg.lg[1] + bg.lg[2]); u += blockDim.x) {
        const int32_t x = (int32_t)(u & ((1u << lgu) - 1u)), r = (int32_t)(u >> lgu);
        const int32_t y = r & ((1 << bg.lg[1]) - 1), z = r >> bg.lg[1];
        if (x >= xus || y >= ext[1] || z >= ext[2]) continue;
        uint32_t* row = grid + ((int64_t)z * bg.dim[1] + y) * row_words;
        if (vec)
            reinterpret_cast<uint4*>(row)[x] = make_uint4(0u, 0u, 0u, 0u);
        else
            row[x] = 0u;
    }
}

// In cleared brick scenes, zeroes the bricks cut into several work items
// (their items OR into the volume), one workgroup a brick, before the fill.
__device__ __forceinline__ void zero_cut_bricks(const TableView& tv, const WorkView& wv) {
    const uint32_t ns = *wv.n_split;
    for (uint32_t j = blockIdx.x; j < ns; j += gridDim.x) {
        const uint32_t gb = wv.split[j];
        const BrickScene& sc = tv.scenes[tv.brick_scene ? tv.brick_scene[gb] : 0u];
        if (sc.flags & kSceneClear) zero_brick(sc, gb - sc.brick_base);
    }
}

// The colscan and base kernels' work for a plain call of few bricks and rows,
// by every workgroup of the scatter for itself: this row's bin offsets from
// the histogram (all of it is read), the cut bricks zeroed, and by workgroup 0
// the words that the fill reads.  False: the records do not fit.
//
// Two launches of latency (5 to 7 us each) for the reading of rows x bricks
// words by every workgroup.  Measured per call with against without, by words:
// 1 M segments in 256^3 (8 K) 79.8 / 89.7 us, 20 000 in 512^3 (10 K) 37.6 / 42.2,
// 100 000 in 512^3 (50 K) 43.3 / 45.6, 300 000 (64 K) 61.4 / 64.8; 100 000 in
// 768^3 (169 K) 90 / 79.
constexpr uint32_t kScanBricks = kHistBlock;    // a thread per brick
constexpr uint32_t kScanWords = 65536;
__device__ __forceinline__ bool scan_in_scatter(const TableView& tv, const BrickScene& sc, const WorkView& wv, uint32_t g,
                                                uint64_t work_bytes, uint32_t* cur) {
    __shared__ uint32_t tot[kScanBricks];
    __shared__ uint64_t lds[kHistBlock / kWave];
    __shared__ uint32_t max_s, busy_s, sample_s[8];
    const uint32_t NB = sc.bg.nbricks, G = sc.rows, t = threadIdx.x;
    if (t < NB) tot[t] = cur[t] = 0u;
    if (t == 0) max_s = busy_s = 0u;
    lds_barrier();
    // Rows c, c + parts, ... of bricks [b, b + per).
    auto sums = [&](auto kPer) {
        constexpr uint32_t per = decltype(kPer)::value;
        typedef uint32_t Words __attribute__((ext_vector_type(per)));
        const uint32_t units = NB / per, parts = (uint32_t)kHistBlock / units, b = t % units, c = t / units;
        if (c >= parts) return;
        const Words* col = reinterpret_cast<const Words*>(wv.hist) + b;
        Words sum = {}, before = {};
#pragma unroll 8
        for (uint32_t r = c; r < G; r += parts) {
            const Words v = col[(size_t)r * units];
            sum += v;
            before += r < g ? v : (Words){};
        }
#pragma unroll
        for (uint32_t i = 0; i < per; ++i) {
            atomicAdd(&tot[per * b + i], sum[i]);
            atomicAdd(&cur[per * b + i], before[i]);
        }
    };
    if (NB % 4u == 0u)
        sums(std::integral_constant<uint32_t, 4>{});
    else
        sums(std::integral_constant<uint32_t, 1>{});
    lds_barrier();
    const uint32_t mine = t < NB ? tot[t] : 0u;
    atomicMax(&max_s, mine);
    const uint64_t busy = __builtin_amdgcn_ballot_w64(mine != 0u);
    if ((t & (kWave - 1)) == 0) atomicAdd(&busy_s, (uint32_t)__popcll(busy));
    uint64_t total;
    const uint64_t base = block_exclusive_sum<kHistBlock>((uint64_t)mine, lds, total);
    if (t < NB) cur[t] += (uint32_t)base;
    const uint64_t cap = work_bytes > wv.rec_off ? (work_bytes - wv.rec_off) / sizeof(Piece) : 0u;
    const bool fits = total <= cap && total < 0xFFFFFFFFull;
    // (Both complete: the sum has barriers.  All workgroups take the same sample.)
    const uint64_t T = cut_threshold(tv, total, max_s, sample_s, [&] { return busy_s; });
    const bool cut = (uint64_t)max_s > T;
    if (cut && fits && (sc.flags & kSceneClear))
        for (uint32_t i = blockIdx.x; i < NB; i += gridDim.x)
            if ((uint64_t)tot[i] > T) zero_brick(sc, i);
    if (blockIdx.x == 0) {
        // Extra items, and above them the cut bricks.
        const uint32_t more = t < NB ? brick_items(mine, T) - 1u : 0u;
        uint64_t extra = 0, first = 0;
        if (cut) first = block_exclusive_sum<kHistBlock>((more ? uint64_t(1) << 32 : 0u) | more, lds, extra);
        if (t < NB) {
            wv.bin_base[t] = (uint32_t)base;
            if (cut) {
                wv.item_base[t] = (uint32_t)first;
                for (uint32_t j = 0; j < more && fits; ++j) wv.item_brick[(uint32_t)first + j] = t;
            }
        }
        if (t == 0) {
            wv.bin_base[NB] = (uint32_t)total;
            *wv.pieces = total;
            if (!fits) *wv.direct_all = 1u;
            if (cut) wv.item_base[NB] = (uint32_t)extra;
            *wv.n_items = cut ? (((uint32_t)extra + 1u) & ~1u) + NB : NB;
            *wv.n_split = (uint32_t)(extra >> 32);
        }
    }
    return fits;
}

template <bool kScan>
__global__ __launch_bounds__(kHistBlock) void k_brick_scatter(uint8_t* __restrict__ work, uint64_t work_bytes) {
    extern __shared__ uint32_t cur[];
    __shared__ Stage<kStage> st;
    const TableView tv = table_view(work + kWorkTable);
    const WorkView wv = work_of(work, tv);
    const uint32_t r = xcd_row(blockIdx.x, gridDim.x);
    if (*wv.ok == 0) return;
    if constexpr (!kScan) {
        if (*wv.direct_all != 0) return;
        zero_cut_bricks(tv, wv);
        if (r >= tv.h.rows) return;
    }
    const BrickScene sc = tv.scenes[!kScan && tv.row_scene ? tv.row_scene[r] : 0u];
    const BrickGeom& bg = sc.bg;
    const uint32_t NB = bg.nbricks;
    const uint32_t g = r - sc.row_base;
    if constexpr (kScan) {
        // (As many workgroups as rows.)
        if (!scan_in_scatter(tv, sc, wv, r, work_bytes, cur) || r >= tv.h.rows) return;
    } else {
        const uint32_t* row = wv.hist + sc.hist_off + (size_t)g * NB;
        const uint32_t* base_b = wv.bin_base + sc.brick_base;
        for (uint32_t b = threadIdx.x; b < NB; b += kHistBlock) cur[b] = base_b[b] + row[b];
    }
    int64_t lo, hi;
    seg_range(sc.n, (int)g, (int)sc.rows, lo, hi);
    Piece* __restrict__ recs = wv.recs;
    const bool euclid = (sc.flags & kSceneEuclid) != 0;
    bool bad = false;
    for (int64_t base = lo; base < hi; base += kStage) {
        const uint32_t cnt = (uint32_t)(hi - base < kStage ? hi - base : kStage);
        stage_segments(sc.segs, base, cnt, bg, euclid, st, nullptr, bad,
                       [](const Seg&, uint32_t) { return false; });
        auto place = [&](const auto& maker, uint32_t b, uint32_t klo, uint32_t khi, int32_t bx, int32_t by,
                         int32_t bz) {
            const uint32_t pos = atomicAdd(&cur[b], 1u);
            recs[pos] = maker(klo, khi, bx, by, bz, bg);
        };
        if (euclid)
            walk_ordered<true, PieceMakerEuclid>(st, bg, true, place);
        else
            walk_ordered<true, PieceMaker>(st, bg, false, place);
        lds_barrier();
    }
    if (bad) atomicOr(wv.status, kStatusOutOfRange);
}

// ------------------------------------------------------------------- fill

template <int LGX, int LGY, int LGZ>
struct BrickShape {
    static constexpr int kBXw = 1 << (LGX - 5);                       // words per row
    static constexpr uint32_t kWords = (uint32_t)kBXw << (LGY + LGZ);
    static constexpr size_t kBytes = (size_t)kWords * 4;
    static constexpr int kMaxLg = LGX > LGY ? (LGX > LGZ ? LGX : LGZ) : (LGY > LGZ ? LGY : LGZ);
};

// The word of a piece record that holds its bit index and length.
template <int LGX, int LGY, int LGZ>
struct RecordBits {
    static constexpr int kIdxBits = LGX + LGY + LGZ;
    static constexpr uint32_t kIdxMask = (1u << kIdxBits) - 1u;
    static_assert(kIdxBits <= 20 && BrickShape<LGX, LGY, LGZ>::kMaxLg <= 8,
                  "bit index, length (8 bits, 9 with the Euclidean N) and axis share a word");
};

// Word of the LDS brick holding bit index idx.  A valid piece stays inside
// its brick; the mask keeps every LDS access inside the brick whatever a
// record holds (the address computation needs a mask anyway, so this costs
// no instruction).
template <int LGX, int LGY, int LGZ>
__device__ __forceinline__ uint32_t brick_word(int32_t idx) {
    return ((uint32_t)idx >> 5) & (BrickShape<LGX, LGY, LGZ>::kWords - 1u);
}

// Most samples of one piece.  A piece lies in one brick.  With the Chebyshev
// N its dominant coordinate moves by one voxel per k, so it has at most as
// many samples as the brick's longest side L.  With the Euclidean N
// (N <= sqrt(3) a_m) the dominant coordinate moves by more than
// (khi - klo) a_m / N - 1 between klo and khi and by at most L - 1 inside
// the brick, so khi - klo < sqrt(3) L and a piece has at most 7L/4 samples
// (L >= 32).
template <bool kEuclid, int LGX, int LGY, int LGZ>
struct MaxSamples {
    static constexpr uint32_t kSide = 1u << BrickShape<LGX, LGY, LGZ>::kMaxLg;
    static constexpr uint32_t kValue = kEuclid ? kSide * 7u / 4u : kSide;
    static_assert(kSide >= 32, "7L/4 bounds sqrt(3) L + 1");
};

// Samples of a piece record (from its last word); a record outside the
// bound above (which the scatter never writes) counts as empty, so that
// every loop of the fill stays bounded whatever the workspace holds.
template <bool kEuclid, int LGX, int LGY, int LGZ>
__device__ __forceinline__ uint32_t record_length(uint32_t w) {
    const uint32_t len = ((w >> RecordBits<LGX, LGY, LGZ>::kIdxBits) & (kEuclid ? 511u : 255u)) + 1u;
    return len <= MaxSamples<kEuclid, LGX, LGY, LGZ>::kValue ? len : 0u;
}

constexpr int kFillChunk = 32;  // samples per chunk
constexpr uint32_t kPairItems = 8;  // items a workgroup from which the queues deal units of two

// Signed strides of the minor axes a < b and of the dominant axis m inside
// the brick, by m | nega << 2 | negb << 3 | negm << 4: a table of 32 entries
// (a, b, m, unused) in LDS.
template <int LGX, int LGY>
__device__ __forceinline__ void make_strides(int4* strides) {
    const uint32_t i = threadIdx.x;
    if (i >= 32u) return;
    const uint32_t m = i & 3u;
    const int32_t x = 1, y = 1 << LGX, z = 1 << (LGX + LGY);
    const int32_t a = m == 0u ? y : x, b = m == 2u ? y : z, d = m == 0u ? x : (m == 1u ? y : z);
    strides[i] = make_int4((i & 4u) ? -a : a, (i & 8u) ? -b : b, (i & 16u) ? -d : d, 0);
}

// Stepping state of a chunk: samples koff ... of the record's piece.  Per
// minor axis a 32-bit fraction f and its slope d: the axis advances at a step
// exactly when f + d carries out of 32 bits (fix23_fraction, the 23-bit fractions
// moved to the top).  A step is five VALU instructions (two adds with carry,
// two selects of a stride, one three-way add of the bit index) and three for
// the LDS word and the bit.  Moving on to a chunk's first sample is a
// multiply-add per axis, where exact remainders (16-bit halves below 2N, the
// form before this one) took a division per axis.
struct StepCheb {
    uint32_t fa, fb, da, db;
    int32_t idx, s0, s1, sb;

    template <int LGX, int LGY, int LGZ>
    __device__ __forceinline__ void start(const u32x4& rec, uint32_t koff, const int4* strides) {
        const int4 st = strides[((rec.z & 32u) >> 1) | (rec.w >> 28)];
        const int32_t sa = st.x, sm = st.z;
        sb = st.y;
        const uint32_t ib = (rec.x & 511u) | ((rec.y & 511u) << 9) | ((rec.z & 31u) << 18);
        const uint32_t ta = __umul24(rec.z >> 9, koff) + (rec.x >> 9);  // below 2^31: koff < 256
        const uint32_t tb = __umul24(ib, koff) + (rec.y >> 9);
        fa = ta << 9;
        fb = tb << 9;
        da = rec.z & ~511u;
        db = ib << 9;
        idx = (int32_t)(rec.w & RecordBits<LGX, LGY, LGZ>::kIdxMask) + __mul24((int32_t)koff, sm) +
              __mul24((int32_t)(ta >> 23), sa) + __mul24((int32_t)(tb >> 23), sb);
        s0 = sm;
        s1 = sm + sa;
    }
    __device__ __forceinline__ void next() {
        const bool ca = __builtin_uadd_overflow(fa, da, &fa);
        const bool cb = __builtin_uadd_overflow(fb, db, &fb);
        idx += (ca ? s1 : s0) + (cb ? sb : 0);
        // (Opaque to the loop optimiser, which would add the slopes a second
        // time in induction variables of their own.)
        asm volatile("" : "+v"(fa), "+v"(fb));
    }
};

// The same under the Euclidean N of eq. (1), where the dominant axis moves
// only when its own fraction carries, and a step that moves no axis sets the
// same bit again.  The record holds integers, so a chunk starts with one
// division per axis at k = klo + koff (numerators below 2^31); the quotients
// move the bit index from the segment's start point, mod the brick's voxel
// count.  Fractions and slopes of 32 bits from the reciprocal (fix32_about).
struct StepEuclid {
    uint32_t f[3], d[3];
    int32_t idx, s[3];

    template <int LGX, int LGY, int LGZ>
    __device__ __forceinline__ void start(const u32x4& rec, uint32_t koff, const int4* strides) {
        const int4 st = strides[rec.z & 31u];
        s[0] = st.x;
        s[1] = st.y;
        s[2] = st.z;
        const uint32_t two_n = rec.z >> 16 > 1u ? rec.z >> 16 : 2u;
        const uint32_t two_a[3] = {rec.y & 0xFFFFu, rec.y >> 16, rec.x >> 16};
        const uint32_t k = (rec.x & 0xFFFFu) + koff;
        const float rcp = __builtin_amdgcn_rcpf((float)two_n), rcpd = rcp_bias_down(rcp);
        const float scale = rcp * 0x1p32f;
        idx = (int32_t)(rec.w & RecordBits<LGX, LGY, LGZ>::kIdxMask);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const uint32_t neg = (rec.z >> (2 + i)) & 1u;
            uint32_t q, r;
            divmod_down(__umul24(k, two_a[i]) + (two_n >> 1) - neg, two_n, rcpd, q, r);
            const bool tie = two_a[i] >= two_n;  // moves at every step
            f[i] = tie ? 0x80000000u : fix32_about(r, scale);
            d[i] = tie ? 0xFFFFFFFFu : fix32_about(two_a[i], scale);
            idx += __mul24((int32_t)q, s[i]);
        }
    }
    __device__ __forceinline__ void next() {
        int32_t mv[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) mv[i] = __builtin_uadd_overflow(f[i], d[i], &f[i]) ? s[i] : 0;
        idx += mv[0] + mv[1] + mv[2];
        asm volatile("" : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]));
    }
};

// Sets the bits of one round: a chunk of n samples per valid lane (lanes in
// descending order of n).  The steps that every valid lane takes run in a
// scalar loop, the few beyond the shortest chunk under the lanes' masks.
template <typename Step, int LGX, int LGY, int LGZ>
__device__ __forceinline__ void run_round(uint32_t* brick, const u32x4& rec, uint32_t koff, uint32_t n,
                                          uint32_t n_min, const int4* strides) {
    Step st;
    st.template start<LGX, LGY, LGZ>(rec, koff, strides);
    uint32_t k = 0;
    auto steps = [&](auto count) {
#pragma unroll
        for (int i = 0; i < decltype(count)::value; ++i) {
            atomicOr(&brick[brick_word<LGX, LGY, LGZ>(st.idx)], 1u << ((uint32_t)st.idx & 31u));
            st.next();
        }
        k += (uint32_t)decltype(count)::value;
    };
    while (k + 8u <= n_min) steps(std::integral_constant<int, 8>{});
    if (k + 4u <= n_min) steps(std::integral_constant<int, 4>{});
    if (k + 2u <= n_min) steps(std::integral_constant<int, 2>{});
    for (; k < n; ++k) {
        atomicOr(&brick[brick_word<LGX, LGY, LGZ>(st.idx)], 1u << ((uint32_t)st.idx & 31u));
        st.next();
    }
}

// Between the kUpr-lane halves of each 2 kUpr lanes: the lower half's value
// for all of them, or the upper half's.
template <int kUpr, bool kUpper>
__device__ __forceinline__ u32x4 swap_rows(const u32x4& v) {
    static_assert(kUpr == 1 || kUpr == 2, "rows of 16 or 32 bytes");
    // quad_perm: [0,1,0,1] / [2,3,2,3], or [0,0,2,2] / [1,1,3,3].
    constexpr int kPerm = kUpr == 2 ? (kUpper ? 0xEE : 0x44) : (kUpper ? 0xF5 : 0xA0);
    const uint32_t x = v.x, y = v.y, z = v.z, w = v.w;
    return (u32x4){(uint32_t)__builtin_amdgcn_mov_dpp((int)x, kPerm, 0xf, 0xf, true),
                   (uint32_t)__builtin_amdgcn_mov_dpp((int)y, kPerm, 0xf, 0xf, true),
                   (uint32_t)__builtin_amdgcn_mov_dpp((int)z, kPerm, 0xf, 0xf, true),
                   (uint32_t)__builtin_amdgcn_mov_dpp((int)w, kPerm, 0xf, 0xf, true)};
}

// The scenes the direct kernel serves: those the brick path does not take
// (flagged by the plan), or every scene when the records did not fit.
// Nothing runs after a failed plan.
__device__ __forceinline__ bool direct_scenes(const uint8_t* work, const TableView& tv, uint32_t& count,
                                              bool& all) {
    const uint32_t* w = reinterpret_cast<const uint32_t*>(work);
    if (w[kWStatus] & (uint32_t)(kStatusInvalid | kStatusLaunch)) return false;
    all = w[kWDirectAll] != 0;
    count = all ? tv.h.n_scenes : tv.h.n_direct;
    return count > 0;
}

// Zeroes the volumes of the cleared direct scenes (whose bits the direct kernel
// sets after the fill).
__device__ __forceinline__ void clear_direct_scenes(const uint8_t* work, const TableView& tv) {
    uint32_t nd;
    bool all;
    if (!direct_scenes(work, tv, nd, all)) return;
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t ts = (int64_t)gridDim.x * blockDim.x;
    for (uint32_t j = 0; j < nd; ++j) {
        const BrickScene& sc = tv.scenes[all ? j : tv.direct[j]];
        if (!(sc.flags & kSceneClear)) continue;
        const int64_t nwords = ((int64_t)sc.bg.dim[0] * sc.bg.dim[1] * sc.bg.dim[2] + 31) / 32;
        clear_words(sc.grid, nwords, t0, ts);
    }
}

// Launch shape of the fill kernel: kWgs workgroups per CU, of 1024 threads
// (one per CU) or 512 (two per CU).  A 128 KiB brick takes a whole CU; 64 KiB
// bricks run either way: two workgroups per CU, so that one workgroup's brick
// start and flush overlap the other's voxel work, or, when the volume has
// fewer bricks than that gives slots, one with all 16 waves on its brick.
//
// The chunk table (16-bit entries: record within the pass | chunk << 12)
// takes the LDS the brick leaves; a pass covers up to kPer records a thread,
// or one a thread when their chunks do not fit the table.
template <int LGX, int LGY, int LGZ, int kWgs>
struct FillCfg {
    static_assert(kWgs == 1 || (kWgs == 2 && LGX + LGY + LGZ < 20), "two workgroups per CU: 64 KiB bricks");
    static constexpr int kBlock = kWgs == 1 ? 1024 : 512;
    static constexpr int kWgsPerCu = kWgs;
    static constexpr int kPer = 3;
    static constexpr int kMaxChunks =
        ((int)MaxSamples<true, LGX, LGY, LGZ>::kValue + kFillChunk - 1) / kFillChunk;  // of a piece
    static constexpr int kFit = (163840 / kWgs - (int)BrickShape<LGX, LGY, LGZ>::kBytes - 1024) / 2;
    static constexpr int kEntCap = kFit < 15360 ? kFit : 15360;
    static_assert(kEntCap >= kBlock * kMaxChunks, "one record a thread always fits the table");
    static_assert(kPer * kBlock <= 4096 && kMaxChunks <= 16, "16-bit chunk entries");
};

// Length words of the records lo + t, lo + t + kBlock, ... of a pass.
template <int kBlock, int kPer>
__device__ __forceinline__ void load_lengths(const uint32_t* __restrict__ recw, uint32_t lo, uint32_t records,
                                             uint32_t w[kPer]) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const uint32_t at = threadIdx.x + (uint32_t)(i * kBlock);
        w[i] = at < records ? recw[4u * ((size_t)lo + at) + 3u] : 0u;
    }
}

// Cutting the pieces of a pass into chunks of at most kFillChunk samples and
// listing them by length, longest first (a counting sort over the lengths in
// LDS), so that a round's 64 chunks have (nearly) equal lengths and the last
// rounds of the brick are the short ones.  count() counts the chunks (bin 0
// the full ones, bin kFillChunk - l the last chunks of l samples) while the
// item before still runs; list() writes the table, after a barrier.
template <int LGX, int LGY, int LGZ, int kWgs>
struct ChunkList {
    using Cfg = FillCfg<LGX, LGY, LGZ, kWgs>;
    static constexpr int kBlock = Cfg::kBlock, kPer = Cfg::kPer;
    uint32_t lr[kPer];  // of the records lo + t, lo + t + kBlock, ...: length | rank in its bin << 16
    uint32_t base;      // this thread's first entry among the full chunks

    // w: length words of the records below hi - lo.
    __device__ __forceinline__ void count(uint32_t* bins, const uint32_t* w, uint32_t records, bool euclid) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const uint32_t len = euclid ? record_length<true, LGX, LGY, LGZ>(w[i])
                                        : record_length<false, LGX, LGY, LGZ>(w[i]);
            lr[i] = threadIdx.x + (uint32_t)(i * kBlock) < records ? len : 0u;
        }
        rank(bins);
    }
    __device__ __forceinline__ void rank(uint32_t* bins) {
        uint32_t full = 0;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const uint32_t l = lr[i] % kFillChunk;
            full += lr[i] / kFillChunk;
            if (l) lr[i] |= atomicAdd(&bins[kFillChunk - l], 1u) << 16;
        }
        const uint32_t incl = wave_inclusive_sum_dpp(full);
        base = 0;
        if (__lane_id() == kWave - 1) base = atomicAdd(&bins[0], incl);
        base = __builtin_amdgcn_readlane(base, kWave - 1) + incl - full;
    }
    // Entries of the table (complete after the next barrier); `records` of
    // the pass shrinks to one a thread when their chunks overflow the table.
    __device__ __forceinline__ uint32_t list(uint16_t* ent, uint32_t* bins, uint32_t& records) {
        const uint32_t lane = __lane_id();
        for (;;) {
            const uint32_t c = lane < (uint32_t)kFillChunk ? bins[lane] : 0u;
            const uint32_t bin_end = wave_inclusive_sum_dpp(c);
            const uint32_t total = __builtin_amdgcn_readlane(bin_end, kWave - 1);
            if (total <= (uint32_t)Cfg::kEntCap) {
                const int bin_start = (int)(bin_end - c);
#pragma unroll
                for (int i = 0; i < kPer; ++i) {
                    const uint32_t len = lr[i] & 0xFFFFu, l = len % kFillChunk, nf = len / kFillChunk;
                    const uint32_t e = threadIdx.x + (uint32_t)(i * kBlock);
                    for (uint32_t j = 0; j < nf; ++j) ent[base + j] = (uint16_t)(e | (j << 12));
                    base += nf;
                    const uint32_t at =
                        (uint32_t)__builtin_amdgcn_ds_bpermute((int)((kFillChunk - l) << 2), bin_start);
                    if (l) ent[at + (lr[i] >> 16)] = (uint16_t)(e | (nf << 12));
                }
                return total;
            }
            lds_barrier();
            if (threadIdx.x < (uint32_t)kFillChunk) bins[threadIdx.x] = 0u;
            lds_barrier();
            records = (uint32_t)kBlock;  // (more than that overflowed the table)
            lr[0] &= 0xFFFFu;
#pragma unroll
            for (int i = 1; i < kPer; ++i) lr[i] = 0u;
            rank(bins);
            lds_barrier();
        }
    }
};

// The rounds of a pass: 64 chunks of the table each, one a lane, claimed by
// the waves in order (the first two of each wave without a claim).  A round
// is claimed, and its records loaded, two rounds before it runs.
template <int kWaves>
struct RoundQueue {
    uint32_t r[2], e[2];
    u32x4 rec[2];

    __device__ __forceinline__ void load(int i, const uint16_t* ent, const u32x4* recp, uint32_t total) {
        const uint32_t c = r[i] * kWave + __lane_id();
        if (c < total) {
            e[i] = ent[c];
            rec[i] = recp[e[i] & 4095u];
        }
    }
    __device__ __forceinline__ void open(const uint16_t* ent, const u32x4* recp, uint32_t total) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            r[i] = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x / kWave) + (uint32_t)(i * kWaves);
            load(i, ent, recp, total);
        }
    }
    // Every wave calls meanwhile() once, after its first round.
    template <int LGX, int LGY, int LGZ, typename F>
    __device__ __forceinline__ void run(uint32_t* brick, const uint16_t* ent, uint32_t* claim_s, const int4* strides,
                                        const u32x4* recp, uint32_t total, bool euclid, F meanwhile) {
        const uint32_t lane = __lane_id();
        for (bool first = true;; first = false) {
            const bool runs = r[0] * kWave < total;
            if (runs) {
                const u32x4 cur = rec[0];
                const uint32_t ce = e[0], c0 = r[0] * kWave;
                r[0] = r[1];
                e[0] = e[1];
                rec[0] = rec[1];
                uint32_t nr = 0;
                if (lane == 0) nr = atomicAdd(claim_s, 1u);
                r[1] = __builtin_amdgcn_readfirstlane(nr);
                load(1, ent, recp, total);
                const uint32_t koff = (ce >> 12) * (uint32_t)kFillChunk;
                const uint32_t len = euclid ? record_length<true, LGX, LGY, LGZ>(cur.w)
                                            : record_length<false, LGX, LGY, LGZ>(cur.w);
                const uint32_t n = len - koff < (uint32_t)kFillChunk ? len - koff : (uint32_t)kFillChunk;
                const uint32_t left = total - c0;
                const uint32_t n_min =
                    __builtin_amdgcn_readlane(n, left < (uint32_t)kWave ? (int)left - 1 : kWave - 1);
                if (lane < left) {
                    if (euclid)
                        run_round<StepEuclid, LGX, LGY, LGZ>(brick, cur, koff, n, n_min, strides);
                    else
                        run_round<StepCheb, LGX, LGY, LGZ>(brick, cur, koff, n, n_min, strides);
                }
            }
            if (first) meanwhile();
            if (!runs) break;
        }
    }
};

// Persistent fill.  Workgroups take work items (a brick, or part of a cut
// brick) from the work queues (work stealing: bricks differ a lot in work).
// The item's pieces are listed as chunks of equal lengths (ChunkList) and
// the waves take rounds of 64 of them from that one list, so that they finish
// a brick together; each lane reads its chunk's record from the L2.  While
// an item's rounds run, the next item is claimed and its records' lengths are
// loaded; its chunks are listed, and each wave's first records loaded, before
// the flush's stores, since a wait for a load also waits for every store
// issued before it.
//
// Bound: in the rounds VALU issue and LDS atomics (8 instructions and one
// atomic a voxel; about half the time), then the write of the volume.  One
// list for the whole workgroup replaces groups of 128 records per wave (their
// chunks in four length classes within the group, digests passed between lanes
// by ds_bpermute), and rows are written in pairs (see the flush): 4 M segments
// of up to 2048 voxels into 2048^3 (19.0 M records, 721.7 M voxels, 1 GiB)
// 0.61 -> 0.47 ms, VALU wave instructions 227 -> 169 M; 100 000 into 512^3
// 20.1 -> 13.4 us.
template <int LGX, int LGY, int LGZ, int kWgs>
__global__ __launch_bounds__((FillCfg<LGX, LGY, LGZ, kWgs>::kBlock), 4)  // 16 waves a CU
void k_brick_fill(uint8_t* __restrict__ work) {
    using Shape = BrickShape<LGX, LGY, LGZ>;
    using Cfg = FillCfg<LGX, LGY, LGZ, kWgs>;
    constexpr int kBlock = Cfg::kBlock, kPer = Cfg::kPer;
    constexpr int kWaves = kBlock / kWave;
    constexpr int kUpr = Shape::kBXw / 4;  // 16-byte units per brick row
    // The brick first, so its addresses need no base offset.
    __shared__ __align__(16) uint32_t brick[Shape::kWords];
    __shared__ uint16_t ent[Cfg::kEntCap];  // chunk table
    __shared__ int4 strides[32];
    __shared__ uint32_t bins[2][kFillChunk];
    __shared__ uint32_t claim_s;
    __shared__ uint32_t next_s[2][4];

    const TableView tv = table_view(work + kWorkTable);
    const WorkView wv = work_of(work, tv);
    if (*wv.direct_all != 0 || tv.h.n_direct != 0) clear_direct_scenes(work, tv);
    if (*wv.ok == 0 || *wv.direct_all != 0) return;
    const uint32_t NB = tv.h.bricks;  // global bricks of all scenes
    FillQueue q;
    q.counter = wv.counter;
    q.items = *wv.n_items;
    q.extra = q.items - NB;
    q.cut = *wv.n_split != 0u;
    // Units of two while every workgroup still gets at least four of them:
    // they halve the partial writes (2048^3: 0.84 against 1.06 ms a call).  With
    // fewer the coarser shares cost more, except where all bricks are alike (at
    // least two of them: 12 wireframes in 512^3 151 against 147 us, 400 000
    // segments in 1024^3 434 against 419, 143 small scenes 450 against 426, but
    // eight wireframes 112.5 against 118).
    const bool two = q.items >= kPairItems * gridDim.x;
    q.units = two ? (q.items + 1u) >> 1 : q.items;
    q.lg = two ? 2u : 3u;
    q.xcd = blockIdx.x % (uint32_t)kXcds;
    q.wgs = gridDim.x;
    uint32_t second = q.items;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const u32x4* recv = reinterpret_cast<const u32x4*>(wv.recs);
    const uint32_t* recw = reinterpret_cast<const uint32_t*>(wv.recs);

    auto scene_of = [&](uint32_t b) {
        return tv.scenes + (tv.brick_scene ? load_uniform(tv.brick_scene + b) : 0u);
    };
    auto euclidean = [&](uint32_t b) { return (load_uniform(&scene_of(b)->flags) & kSceneEuclid) != 0u; };
    auto hand_over = [&](const ItemClaim& c, uint32_t p) {  // (every lane writes the same)
        next_s[p][0] = c.brick;
        next_s[p][1] = c.lo;
        next_s[p][2] = c.hi;
        next_s[p][3] = c.split;
    };
    auto take_over = [&](uint32_t p) {
        return ItemClaim{(uint32_t)__builtin_amdgcn_readfirstlane(next_s[p][0]),
                         (uint32_t)__builtin_amdgcn_readfirstlane(next_s[p][1]),
                         (uint32_t)__builtin_amdgcn_readfirstlane(next_s[p][2]),
                         (uint32_t)__builtin_amdgcn_readfirstlane(next_s[p][3])};
    };
    auto claim = [&]() { return claim_item(wv, q, NB, second); };

    if (wave == 0u) hand_over(claim_item(wv, q, NB, second, true), 0u);
    if (threadIdx.x < (uint32_t)kFillChunk) bins[0][threadIdx.x] = bins[1][threadIdx.x] = 0u;
    make_strides<LGX, LGY>(strides);
    {
        u32x4* b4 = reinterpret_cast<u32x4*>(brick);
        for (uint32_t w = threadIdx.x; w < Shape::kWords / 4; w += kBlock) b4[w] = (u32x4){0, 0, 0, 0};
    }
    lds_barrier();
    ItemClaim it = take_over(0u);
    if (it.brick >= NB) return;

    // A brick waiting for its neighbour along x (see the flush).
    constexpr int kHold = (int)(Shape::kWords / 4) / kBlock;
    u32x4 held[kHold];
    bool holds = false;

    uint32_t w[kPer];
    ChunkList<LGX, LGY, LGZ, kWgs> list;
    auto pass_records = [&](uint32_t lo, uint32_t hi) {
        return hi - lo < (uint32_t)(kPer * kBlock) ? hi - lo : (uint32_t)(kPer * kBlock);
    };
    // The pass that runs: records [lo, lo + records) of item `it`.
    uint32_t lo = it.lo, records = pass_records(lo, it.hi);
    bool euclid = euclidean(it.brick);
    load_lengths<kBlock, kPer>(recw, lo, records, w);
    if (wave == 0u) hand_over(claim(), 1u);
    list.count(bins[0], w, records, euclid);
    lds_barrier();
    // The pass after it.
    ItemClaim nx;
    uint32_t nlo, nrecords;
    bool last, more, next_euclid;
    RoundQueue<kWaves> rounds;
    uint32_t p = 1u;       // the next pass is counted in bins[p]
    uint32_t ip = 1u;      // the next item is in next_s[ip]
    uint32_t chunks;
    // Writes the pass's chunk table (its chunks are counted) and loads what
    // the rounds read first, and the lengths of the pass after it.
    auto open_pass = [&]() {
        chunks = list.list(ent, bins[p ^ 1u], records);
        if (threadIdx.x == 0) claim_s = 2u * (uint32_t)kWaves;
        lds_barrier();
        if (threadIdx.x < (uint32_t)kFillChunk) bins[p ^ 1u][threadIdx.x] = 0u;  // (read before the barrier)
        rounds.open(ent, recv + lo, chunks);
        last = lo + records == it.hi;
        nx = it;
        if (last) {
            nx = take_over(ip);
            ip ^= 1u;
        }
        nlo = last ? nx.lo : lo + records;
        more = nx.brick < NB;
        nrecords = more ? pass_records(nlo, nx.hi) : 0u;
        load_lengths<kBlock, kPer>(recw, nlo, nrecords, w);
        next_euclid = more && euclidean(nx.brick);
    };
    open_pass();

    for (;;) {
        // (The brick is zero: done before the barrier that ended the last item.)
        rounds.template run<LGX, LGY, LGZ>(brick, ent, &claim_s, strides, recv + lo, chunks, euclid, [&]() {
            list.count(bins[p], w, nrecords, next_euclid);
            if (wave == 0u && last && more) hand_over(claim(), ip);
        });
        lds_barrier();  // every wave done with the pass, and the next one counted
        const ItemClaim done = it;
        const bool flush = last, ends = !more;
        if (more) {
            it = nx;
            lo = nlo;
            records = nrecords;
            euclid = next_euclid;
            p ^= 1u;
            open_pass();
        }
        if (flush) {
        // The brick's scene and its place in that scene's volume.
        const BrickScene sc = load_uniform(scene_of(done.brick));
        const BrickGeom bg = sc.bg;
        uint32_t* __restrict__ grid = sc.grid;
        const bool clear = (sc.flags & kSceneClear) != 0;
        const uint32_t lb = done.brick - sc.brick_base;
        const int64_t row_words = (int64_t)bg.dim[0] >> 5;
        const int bx = (int)(lb % (uint32_t)bg.nb[0]);
        const int by = (int)((lb / (uint32_t)bg.nb[0]) % (uint32_t)bg.nb[1]);
        const int bz = (int)(lb / ((uint32_t)bg.nb[0] * (uint32_t)bg.nb[1]));
        const int32_t org[3] = {bx << LGX, by << LGY, bz << LGZ};
        int32_t ext[3];
        {
            const int lgs[3] = {LGX, LGY, LGZ};
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                const int32_t x = bg.dim[ax] - org[ax];
                ext[ax] = x < (1 << lgs[ax]) ? x : (1 << lgs[ax]);
            }
        }
        // Flush: brick rows -> volume words, zeroing the brick on the way.
        // The owner of a whole brick writes every word of it, so a clearing
        // call needs no other pass.  A brick with no pieces in a scene that
        // ORs into its volume changes nothing: no flush (its LDS copy is
        // still zero).  An item holding part of a cut brick ORs its nonzero
        // words into the volume with device atomics (the other items of the
        // brick do the same; the scatter zeroed the brick first in a cleared
        // volume).
        //
        // Rows of 32 bytes written alone reach HBM as partial 64-byte blocks
        // once the workgroups' flushes no longer coincide: writing 1 GiB in
        // 256x64x64 bricks with 8 us of other work per brick takes 0.74 ms,
        // against 0.40 ms when the bricks' rows are written in pairs side by
        // side.  So a brick whose right neighbour is this workgroup's next
        // item waits in registers (32 VGPRs) and is stored with it.
        const bool exists = lb < bg.nbricks;
        const int rows = exists && (clear || done.lo != done.hi) ? ext[1] * ext[2] : 0;
        // Whole 16-byte units when the volume's rows hold whole brick rows.
        const bool vec = Shape::kBXw % 4 == 0 && (bg.dim[0] & ((1 << LGX) - 1)) == 0;
        const bool full_y = ext[1] == (1 << LGY);  // rows per slab a power of two
        const bool whole = vec && full_y && !done.split;
        if (whole && !holds && rows != 0 && !ends && it.brick == done.brick + 1u && !it.split && bx + 1 < bg.nb[0]) {
            u32x4* src = reinterpret_cast<u32x4*>(brick) + threadIdx.x;
#pragma unroll
            for (int i = 0; i < kHold; ++i) {
                held[i] = src[i * kBlock];
                src[i * kBlock] = (u32x4){0u, 0u, 0u, 0u};
            }
            holds = true;
        } else if (done.split) {
            // By shifts, over the rows as wide as the next power of two (words
            // outside the volume are zero; divisions by the extents took a part some
            // 20 us), neighbouring lanes neighbouring words (four words a lane: twice
            // the time where most are set).
            const int xws = ext[0] >> 5, lgx = xws > 1 ? 32 - __builtin_clz((uint32_t)xws - 1u) : 0;
            const int total = (ext[2] << LGY) << lgx;
            uint32_t* dst = grid + ((int64_t)org[2] * bg.dim[1] + org[1]) * row_words + (org[0] >> 5);
            constexpr int kAtOnce = 8;
            for (int t = threadIdx.x; t < total; t += kBlock * kAtOnce) {
                // (Beyond the last word that one is read, and not flushed again:
                // hundreds of atomics on one word.)
                uint32_t v[kAtOnce];
                auto word = [&](int w) { return brick + ((w >> lgx) * Shape::kBXw + (w & ((1 << lgx) - 1))); };
#pragma unroll
                for (int j = 0; j < kAtOnce; ++j) v[j] = *word(t + j * kBlock < total ? t + j * kBlock : total - 1);
#pragma unroll
                for (int j = 0; j < kAtOnce; ++j) {
                    const int w = t + j * kBlock, r = w >> lgx;
                    if (w >= total || v[j] == 0u) continue;
                    *word(w) = 0u;  // zero for the next item
                    __hip_atomic_fetch_or(dst + ((int64_t)(r >> LGY) * bg.dim[1] + (r & ((1 << LGY) - 1))) * row_words +
                                              (w & ((1 << lgx) - 1)),
                                          v[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        } else if (whole) {
            // 16-byte units, kUpr per row, rows full width and full slabs:
            // a thread's units share their row in the slab and their part of
            // the row, and step by a fixed number of slabs (kBlock units are
            // a whole number of slabs in every compiled shape).
            constexpr int kRowsPerStep = kBlock / kUpr;
            static_assert(kBlock % kUpr == 0 && kRowsPerStep % (1 << LGY) == 0, "whole slabs per step");
            constexpr int kSlabsPerStep = kRowsPerStep >> LGY;
            const int units = (holds ? ext[1] * ext[2] : rows) * kUpr;
            const int part = (int)threadIdx.x % kUpr, r0 = (int)threadIdx.x / kUpr;
            const int y = r0 & ((1 << LGY) - 1), z0 = r0 >> LGY;
            u32x4* src = reinterpret_cast<u32x4*>(brick) + threadIdx.x;
            global_u32x4* dst = (global_u32x4*)(
                grid + ((int64_t)(org[2] + z0) * bg.dim[1] + (org[1] + y)) * row_words + (org[0] >> 5) + 4 * part);
            const int64_t dst_step = (int64_t)kSlabsPerStep * bg.dim[1] * row_words / 4;  // in 16-byte units
            if (holds) {
                // The rows of this brick and of the held one, side by side:
                // lanes of a pair of rows exchange units, so that 2 kUpr
                // lanes write the 32 kUpr bytes of one row.
                const bool hi = ((int)threadIdx.x & kUpr) != 0;
                dst = dst - kUpr - (hi ? row_words / 4 : 0) + (hi ? kUpr : 0);
#pragma unroll
                for (int i = 0; i < kHold; ++i) {
                    if ((int)threadIdx.x + i * kBlock < units) {
                        const u32x4 v = src[i * kBlock];
                        src[i * kBlock] = (u32x4){0u, 0u, 0u, 0u};  // zero for the next item
                        // (Exchanged by all lanes, then selected.)
                        const u32x4 lower = swap_rows<kUpr, false>(v), upper = swap_rows<kUpr, true>(held[i]);
                        u32x4 r0 = hi ? lower : held[i], r1 = hi ? v : upper;
                        if (!clear) {
                            r0 |= dst[0];
                            r1 |= dst[row_words / 4];
                        }
                        // (Whole 64-byte blocks: past the caches, which the
                        // records need.  2048^3: 0.837 against 0.905 ms.)
                        __builtin_nontemporal_store(r0, dst);
                        __builtin_nontemporal_store(r1, dst + row_words / 4);
                    }
                    dst += dst_step;
                }
            } else {
#pragma unroll
                for (int i = 0; i < kHold; ++i) {
                    if ((int)threadIdx.x + i * kBlock < units) {
                        const u32x4 v = src[i * kBlock];
                        src[i * kBlock] = (u32x4){0u, 0u, 0u, 0u};  // zero for the next item
                        *dst = clear ? v : *dst | v;
                    }
                    dst += dst_step;
                }
            }
            holds = false;
        } else if (vec) {
            // 16-byte units, kUpr per row, rows full width.
            const int units = rows * kUpr;
            for (int t = threadIdx.x; t < units; t += kBlock) {
                const int part = t % kUpr, r = t / kUpr;
                const int y = full_y ? (r & ((1 << LGY) - 1)) : r % ext[1];
                const int z = full_y ? (r >> LGY) : r / ext[1];
                u32x4* src = reinterpret_cast<u32x4*>(
                    &brick[(((uint32_t)z << LGY) | (uint32_t)y) * (uint32_t)Shape::kBXw + 4u * part]);
                const u32x4 v = *src;
                *src = (u32x4){0u, 0u, 0u, 0u};  // zero for the next item
                global_u32x4* dst = (global_u32x4*)(
                    grid + ((int64_t)(org[2] + z) * bg.dim[1] + (org[1] + y)) * row_words + (org[0] >> 5) +
                    4 * part);
                if (clear) {
                    *dst = v;
                } else {
                    *dst = *dst | v;
                }
            }
        } else {
            const int xws = ext[0] >> 5;
            const int total = rows * xws;
            for (int t = threadIdx.x; t < total; t += kBlock) {
                const int xw = t % xws, r = t / xws;
                const int y = r % ext[1], z = r / ext[1];
                uint32_t* src = &brick[(((uint32_t)z << LGY) | (uint32_t)y) * (uint32_t)Shape::kBXw + xw];
                const uint32_t v = *src;
                *src = 0u;  // zero for the next item
                global_u32* dst = (global_u32*)grid + ((int64_t)(org[2] + z) * bg.dim[1] + (org[1] + y)) * row_words +
                                (org[0] >> 5) + xw;
                if (clear) *dst = v;
                else *dst |= v;
            }
        }
        // Every word that can hold a bit (inside the volume) was read and
        // zeroed above; the others were never set.
        }
        if (ends) break;
        lds_barrier();
    }
}

// ------------------------------------------------------- direct scenes

constexpr int kDirectBlock = 256;

// The segments of the direct scenes, one device atomic per voxel
// (direct_segments, vox_direct.h; the merge of neighbouring bits that plain calls
// of many segments take has not been measured here).
__global__ __launch_bounds__(kDirectBlock) void k_batch_direct(uint8_t* __restrict__ work) {
    const TableView tv = table_view(work + kWorkTable);
    uint32_t nd;
    bool all;
    if (!direct_scenes(work, tv, nd, all)) return;
    int32_t* status = reinterpret_cast<int32_t*>(work) + kWStatus;
    const int64_t wave0 = (int64_t)blockIdx.x * (kDirectBlock / kWave) + threadIdx.x / kWave;
    const int64_t ws = (int64_t)gridDim.x * (kDirectBlock / kWave);
    for (uint32_t j = 0; j < nd; ++j) {
        const BrickScene sc = tv.scenes[all ? j : tv.direct[j]];
        const int32_t dx = sc.bg.dim[0], dy = sc.bg.dim[1], dz = sc.bg.dim[2];
        const bool a8 = (sc.flags & kSceneA8) != 0;
        if (sc.flags & kSceneEuclid) {
            if (a8)
                direct_segments<true, true>(sc.segs, sc.n, dx, dy, dz, sc.grid, sc.counts, status, wave0, ws);
            else
                direct_segments<false, true>(sc.segs, sc.n, dx, dy, dz, sc.grid, sc.counts, status, wave0, ws);
        } else {
            if (a8)
                direct_segments<true, false>(sc.segs, sc.n, dx, dy, dz, sc.grid, sc.counts, status, wave0, ws);
            else
                direct_segments<false, false>(sc.segs, sc.n, dx, dy, dz, sc.grid, sc.counts, status, wave0, ws);
        }
    }
}

// ---------------------------------------------------------------- host side

// Brick shapes with a compiled fill kernel.
static const int kShapes[][3] = {{8, 6, 5}, {8, 6, 6}, {7, 6, 6}, {7, 7, 6}};

bool brick_shape_supported(const int lg[3]) {
    for (const auto& sh : kShapes)
        if (sh[0] == lg[0] && sh[1] == lg[1] && sh[2] == lg[2]) return true;
    return false;
}

bool brick_geometry_for(int32_t dx, int32_t dy, int32_t dz, const int lg[3], BrickGeom& bg) {
    return brick_geometry(dx, dy, dz, lg, bg);
}

// 256 x 64 x 64 bricks (128 KiB of LDS) when the volume still has at least
// 4096 of them, i.e. 16 per CU for the work stealing to balance; otherwise
// 256 x 64 x 32.  Rows of 256 voxels are 32 bytes, whole memory sectors.
void default_brick_lg(int32_t dx, int32_t dy, int32_t dz, int lg[3]) {
    const int64_t big = ((int64_t)(dx + 255) >> 8) * ((dy + 63) >> 6) * ((dz + 63) >> 6);
    lg[0] = 8;
    lg[1] = 6;
    lg[2] = big >= 4096 ? 6 : 5;
}

// Worst case of pieces: every segment crossing every brick boundary of
// every axis once.
uint64_t max_pieces(int64_t n, const BrickGeom& bg) {
    return (uint64_t)n * (uint64_t)(1 + (bg.nb[0] - 1) + (bg.nb[1] - 1) + (bg.nb[2] - 1));
}

static uint64_t table_bytes(uint32_t n_scenes, uint32_t rows, uint32_t bricks) {
    uint64_t b = kTableScenes + (uint64_t)n_scenes * (sizeof(BrickScene) + 4u);
    if (n_scenes > 1) b += 4ull * ((uint64_t)rows + bricks);
    return up256(b);
}

BrickLaunch batch_launch(uint32_t n_scenes, uint64_t total_segments, const int lg[3]) {
    BrickLaunch L;
    L.n_scenes = n_scenes;
    L.total_segments = total_segments;
    // Rows of scene s: min(256, max(1, ceil(n_s / per_row))) <= 1 + n_s / per_row,
    // with the plain calls' rows of 512 segments for a single scene.
    const uint64_t per_row = n_scenes == 1 ? (uint64_t)kSegsPerRowPlain : (uint64_t)kSegsPerRow;
    uint64_t rows = (uint64_t)n_scenes + (total_segments + per_row - 1) / per_row;
    const uint64_t rmax = (uint64_t)n_scenes * kHistRows;
    L.rows = (uint32_t)(rows < rmax ? rows : rmax);
    L.bricks = (uint32_t)((uint64_t)n_scenes * kMaxBricks);
    for (int a = 0; a < 3; ++a) L.lg[a] = lg[a];
    L.table_bytes = table_bytes(n_scenes, L.rows, L.bricks);
    L.direct_kernels = true;
    L.segs_per_row = (uint32_t)per_row;
    return L;
}

// Table, histograms (each scene's rows times at most kMaxBricks bricks),
// brick totals, offsets and work items.
size_t batch_fixed_bytes(const BrickLaunch& L) {
    return (size_t)(kWorkTable + L.table_bytes + brick_data_bytes((uint64_t)L.rows * kMaxBricks, L.bricks));
}

BrickLaunch plain_launch(int64_t n, const BrickGeom& bg) {
    BrickLaunch L;
    L.n_scenes = 1;
    L.total_segments = (uint64_t)n;
    L.rows = hist_rows(n, kSegsPerRowPlain);
    L.segs_per_row = (uint32_t)kSegsPerRowPlain;
    L.bricks = bg.nbricks;
    for (int a = 0; a < 3; ++a) L.lg[a] = bg.lg[a];
    L.table_bytes = table_bytes(1, L.rows, L.bricks);
    // The caller's workspace holds the worst case of records.
    L.direct_kernels = false;
    return L;
}

size_t brick_workspace_bytes(int64_t n, const BrickGeom& bg) {
    const BrickLaunch L = plain_launch(n, bg);
    return (size_t)(kWorkTable + L.table_bytes + brick_data_bytes((uint64_t)L.rows * bg.nbricks, L.bricks) +
                    max_pieces(n, bg) * sizeof(Piece));
}

static int device_cus() {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
        cus = 256;
    return cus;
}

// Persistent fill workgroups: wgs_per_cu per compute unit (0: for 64 KiB
// bricks two, unless the launch has fewer bricks than two per CU, then one
// of 1024 threads), and no more than the launch can have work items (a
// workgroup without one would only take a CU slot).
template <int LGX, int LGY, int LGZ>
static hipError_t launch_fill(uint8_t* work, int wgs_per_cu, uint32_t max_bricks, hipStream_t stream) {
    const int cus = device_cus();
    int per = 1;
    if constexpr (LGX + LGY + LGZ < 20)
        per = wgs_per_cu == 1 || wgs_per_cu == 2 ? wgs_per_cu : (max_bricks < 2u * (uint32_t)cus ? 1 : 2);
    int wgs = cus * per;
    if ((uint64_t)wgs > (uint64_t)max_bricks + kMaxExtraItems) wgs = (int)(max_bricks + kMaxExtraItems);
    if constexpr (LGX + LGY + LGZ < 20) {
        if (per == 2) {
            k_brick_fill<LGX, LGY, LGZ, 2><<<wgs, FillCfg<LGX, LGY, LGZ, 2>::kBlock, 0, stream>>>(work);
            return hipGetLastError();
        }
    }
    k_brick_fill<LGX, LGY, LGZ, 1><<<wgs, FillCfg<LGX, LGY, LGZ, 1>::kBlock, 0, stream>>>(work);
    return hipGetLastError();
}

hipError_t launch_bricks(const void* d_scenes, const void* one, const BrickLaunch& L, int fill_wgs_per_cu,
                         void* d_work, size_t work_bytes, hipStream_t stream) {
    if (L.n_scenes < 1 || L.rows < 1 || L.bricks < 1 || !brick_shape_supported(L.lg)) return hipErrorInvalidValue;
    uint8_t* work = static_cast<uint8_t*>(d_work);
    hipError_t e;
    {
        static hipError_t attr = [] {
            hipError_t r = hipFuncSetAttribute((const void*)k_brick_plan_hist,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)kHistLds);
            if (r != hipSuccess) return r;
            return hipFuncSetAttribute((const void*)k_brick_scatter<false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)(kMaxBricks * sizeof(uint32_t)));
        }();
        if (attr != hipSuccess) return attr;
    }
    // A plain call (its one scene by value; the brick geometry keeps it to at
    // most kMaxBricks bricks): the plan runs inside the histogram launch, three
    // to five launches in all; a batch (a device scene array) takes seven.
    if (one) {
        if (L.n_scenes != 1 || L.bricks > kMaxBricks) return hipErrorInvalidValue;
        KernelTimer t("brick_plan_hist", stream);
        k_brick_plan_hist<<<L.rows, kHistBlock, kHistLds, stream>>>(*static_cast<const vox_scene*>(one), L, work,
                                                                    (uint64_t)work_bytes);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    } else {
        {
            KernelTimer t("brick_plan", stream);
            auto plan = [&](auto block) {
                constexpr int kBlock = decltype(block)::value;
                k_brick_plan<kBlock><<<1, kBlock, 0, stream>>>(static_cast<const vox_scene*>(d_scenes), L, work,
                                                               (uint64_t)work_bytes);
            };
            // As many threads as scenes, so fewer waves and cheaper scans: 8 scenes
            // 0.0047 ms against 0.0100 with 1024 threads, 256 scenes 0.0075
            // against 0.0135.
            if (L.n_scenes <= 64u)
                plan(std::integral_constant<int, 64>{});
            else if (L.n_scenes <= 256u)
                plan(std::integral_constant<int, 256>{});
            else
                plan(std::integral_constant<int, 1024>{});
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
        {
            KernelTimer t("brick_hist", stream);
            k_brick_hist<<<L.rows, kHistBlock, 0, stream>>>(work);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    // A plain call with few histogram words scans them in the scatter.
    BrickScene plan{};
    if (one) (void)plan_scene(*static_cast<const vox_scene*>(one), L.lg, (int64_t)L.segs_per_row, plan);
    const uint32_t nb = plan.bg.nbricks;
    const bool scan = nb != 0u && nb <= kScanBricks && nb * plan.rows <= kScanWords;
    if (!scan) {
        {
            KernelTimer t("brick_colscan", stream);
            uint32_t blocks = (L.bricks + kColBins - 1) / kColBins;
            if (blocks > kColMaxBlocks) blocks = kColMaxBlocks;
            k_brick_colscan<<<blocks, 256, 0, stream>>>(work);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
        {
            KernelTimer t("brick_base", stream);
            k_brick_base<<<1, kBaseBlock, 0, stream>>>(work, (uint64_t)work_bytes);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    {
        KernelTimer t("brick_scatter", stream);
        const uint32_t counters = scan ? nb : (L.n_scenes > 1 ? kMaxBricks : L.bricks);
        const size_t scatter_lds = (size_t)counters * sizeof(uint32_t);
        if (scan)
            k_brick_scatter<true><<<L.rows, kHistBlock, scatter_lds, stream>>>(work, (uint64_t)work_bytes);
        else
            k_brick_scatter<false><<<L.rows, kHistBlock, scatter_lds, stream>>>(work, (uint64_t)work_bytes);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    {
        KernelTimer t("brick_fill", stream);
        const int* lg = L.lg;
        if (lg[0] == 8 && lg[1] == 6 && lg[2] == 5) e = launch_fill<8, 6, 5>(work, fill_wgs_per_cu, L.bricks, stream);
        else if (lg[0] == 8 && lg[1] == 6 && lg[2] == 6) e = launch_fill<8, 6, 6>(work, fill_wgs_per_cu, L.bricks, stream);
        else if (lg[0] == 7 && lg[1] == 6 && lg[2] == 6) e = launch_fill<7, 6, 6>(work, fill_wgs_per_cu, L.bricks, stream);
        else if (lg[0] == 7 && lg[1] == 7 && lg[2] == 6) e = launch_fill<7, 7, 6>(work, fill_wgs_per_cu, L.bricks, stream);
        else e = hipErrorInvalidValue;
    }
    if (e != hipSuccess) return e;
    if (L.direct_kernels) {
        KernelTimer t("batch_direct", stream);
        k_batch_direct<<<2048, kDirectBlock, 0, stream>>>(work);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace vox
