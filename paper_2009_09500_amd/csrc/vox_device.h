// Device-side building blocks shared by the voxelization kernels (gfx950,
// wave64).  Internal to the HIP library; not part of the C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace vox {

constexpr int kWave = 64;

// Barrier that waits for this wave's LDS traffic only, so global loads
// issued before it (prefetches) stay in flight.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// One segment as read from the caller's AoS array: start point and end
// point.  Loaded with three 8-byte loads when the array is 8-byte aligned
// (every torch allocation is), else six 4-byte loads.
struct Seg {
    int32_t p0[3];
    int32_t p1[3];
};

template <bool kAligned8>
__device__ __forceinline__ Seg load_seg(const int32_t* __restrict__ segs, int64_t i) {
    Seg s;
    const int32_t* p = segs + 6 * i;
    if constexpr (kAligned8) {
        const int2* q = reinterpret_cast<const int2*>(p);
        int2 a = q[0], b = q[1], c = q[2];
        s.p0[0] = a.x; s.p0[1] = a.y; s.p0[2] = b.x;
        s.p1[0] = b.y; s.p1[1] = c.x; s.p1[2] = c.y;
    } else {
        s.p0[0] = p[0]; s.p0[1] = p[1]; s.p0[2] = p[2];
        s.p1[0] = p[3]; s.p1[1] = p[4]; s.p1[2] = p[5];
    }
    return s;
}

// Chebyshev length N = max_a |p1_a - p0_a| in 64 bits (int32 inputs may
// differ by up to 2^32 - 1).
__device__ __forceinline__ int64_t seg_length(const Seg& s) {
    int64_t n = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        int64_t d = (int64_t)s.p1[a] - (int64_t)s.p0[a];
        d = d < 0 ? -d : d;
        n = d > n ? d : n;
    }
    return n;
}

// Euclidean length of the paper's eq. (1), N_e = int(|p1 - p0|): the integer
// square root of dx^2 + dy^2 + dz^2.  For end points within 2^31 of each
// other the sum stays below 2^64 (and below 2^53, where the double square
// root is within one of the result, for every input the library accepts:
// int16 lists, volumes up to 2^20 a side); the integer corrections make it
// exact.
__device__ __forceinline__ uint32_t euclid_length(const Seg& s) {
    uint64_t ss = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int64_t d = (int64_t)s.p1[a] - (int64_t)s.p0[a];
        ss += (uint64_t)(d * d);
    }
    uint64_t r = (uint64_t)sqrt((double)ss);
    while (r * r > ss) --r;
    while ((r + 1) * (r + 1) <= ss) ++r;
    return (uint32_t)r;
}

__device__ __forceinline__ bool in_int16(const Seg& s) {
    bool ok = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        ok &= (s.p0[a] >= -32768) & (s.p0[a] <= 32767) & (s.p1[a] >= -32768) & (s.p1[a] <= 32767);
    }
    return ok;
}

// Domain of the int32 lists: every |p1_a - p0_a| < 2^30, so N < 2^30 and the
// stepping's remainders (below 2N) plus their increments (at most 2N) stay
// below 2^32.
__device__ __forceinline__ bool span_below_2p30(const Seg& s) {
    bool ok = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int64_t d = (int64_t)s.p1[a] - (int64_t)s.p0[a];
        ok &= (d < (int64_t(1) << 30)) & (d > -(int64_t(1) << 30));
    }
    return ok;
}

// Exact incremental evaluation of voxel k of a segment along one axis.
//
// With N the Chebyshev length, d = p1 - p0 and a = |d|, the coordinate is
//   d >= 0:  p0 + floor((2 k a + N) / 2N)
//   d <  0:  p0 - floor((2 k a + N - 1) / 2N)
// (the second is the first with d negated and floor(x + 1/2) mirrored).
// Keeping q = numerator / 2N and r = numerator mod 2N, k -> k + 1 adds 2a
// to the numerator; as 2a <= 2N the quotient grows by at most one:
//   r += 2a;  if (r >= 2N) { r -= 2N; ++q; }
// This is Bresenham's error term; it reproduces the division exactly.
// floor(x / y) and remainder for x < 2^31, 2 <= y < 2^16 and quotients
// below 2^15, from a hardware reciprocal estimate corrected in integers
// (exact).  rcp_down(y) is the reciprocal (within one ulp) scaled by
// 1 - 2^-20: x (rounded once in float) times it is below x / y by a relative
// 2^-20 +- 2^-22, so its integer part is the quotient or one less (the
// quotient is below 2^15, so the shortfall stays below one), and one
// upward correction makes it exact.
//
// The scaling and the division are host+device so that a host program can
// run them with the reciprocal estimate off by -1, 0 and +1 ulp (the
// hardware's stated error), checking the exactness claim on the CPU.
__host__ __device__ __forceinline__ uint32_t mul_u24(uint32_t a, uint32_t b) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __umul24(a, b);
#else
    return (a & 0xFFFFFFu) * (b & 0xFFFFFFu);
#endif
}

__host__ __device__ __forceinline__ float rcp_bias_down(float rcp) { return rcp * (1.0f - 0x1p-20f); }

__device__ __forceinline__ float rcp_down(uint32_t y) {
    return rcp_bias_down(__builtin_amdgcn_rcpf((float)y));
}

__host__ __device__ __forceinline__ void divmod_down(uint32_t x, uint32_t y, float rcpd, uint32_t& q,
                                                     uint32_t& r) {
    uint32_t qq = (uint32_t)((float)x * rcpd);
    uint32_t rr = x - mul_u24(qq, y);
    if (rr >= y) {
        ++qq;
        rr -= y;
    }
    q = qq;
    r = rr;
}

// ceil(x 2^23 / y) for x < y, 2 <= y <= 2^15, from the hardware reciprocal of
// y (within one ulp): the float quotient is within three units, the integer
// remainder to it is exact mod 2^32, and since remainders over y fall on
// multiples of 2^-15, the bias of 2^-17 leaves their ceiling exact.
__host__ __device__ __forceinline__ uint32_t fix23_ceil(uint32_t x, uint32_t y, float rcp) {
    const uint32_t q = (uint32_t)((float)x * (rcp * 0x1p23f));
    const int32_t rem = (int32_t)((x << 23) - mul_u24(q, y));
    return q + (uint32_t)(int32_t)__builtin_ceilf((float)rem * rcp - 0x1p-17f);
}

// One minor axis of a piece in 23-bit fractions: eq. (3)'s quotient advances
// at a step exactly when the fraction's sum passes one.  The fraction is the
// remainder r over 2N at the piece's first voxel, the slope a / N, both
// rounded up, so that after j steps the sum is less than j + 1 units too
// large, and remainders are multiples of 1 / 2N: with j + 1 <= 256 and
// 2N < 2^15 that is below the distance 2^23 / 2N of any fraction to the next
// quotient, so every quotient is exact.  An axis as long as the dominant one
// (two_a = two_n) advances at every step: 1 - 2^-23 a step from the middle.
__host__ __device__ __forceinline__ uint32_t fix23_slope(uint32_t two_a, uint32_t two_n, float rcp) {
    const uint32_t s = fix23_ceil(two_a < two_n ? two_a : 0u, two_n, rcp);
    return two_a < two_n ? s : (1u << 23) - 1u;
}
__host__ __device__ __forceinline__ uint32_t fix23_fraction(uint32_t r, uint32_t two_a, uint32_t two_n, float rcp) {
    const uint32_t f = fix23_ceil(r, two_n, rcp);
    return two_a < two_n ? f : 1u << 22;
}

// Axes under the Euclidean N of eq. (1), where a <= N, as 32-bit fractions: an axis
// moves at a step exactly when fraction and slope carry.
//
// From a remainder r < 2N, and 2a < 2N as its step (lists, whole walks, N <=
// 32767): both rounded up, by less than 1.2 units, so after N steps the sum is less
// than 1.2 (N + 1) <= 2^32 / 2N units too large, and values are multiples of 1 / 2N.
// unit: 2^32 / 2N.
__host__ __device__ __forceinline__ uint32_t fix32_of(uint32_t x, double unit) {
    return (uint32_t)__builtin_ceil((double)x * unit + 0.125);
}
// From the segment (lists, N <= 32767): at sample k the axis has moved the high word
// of fix32_at(k), whose low word is its fraction, in the direction of its sign.  An
// axis with a = N moves at every step: a slope of 1 - 2^-32 from a start of 1/2.
constexpr uint32_t kFix32Always = ~0u;
__host__ __device__ __forceinline__ uint32_t fix32_slope(uint32_t a, uint32_t N, double rcp_n) {
    return a == N ? kFix32Always : (uint32_t)__builtin_ceil((double)a * 0x1p32 * rcp_n + 0.125);
}
// Start of an axis with a negative direction, 1/2 - 1/2N (others 1/2).
__host__ __device__ __forceinline__ uint32_t fix32_start(double rcp_n) {
    return 0x80000000u - (uint32_t)(0x1p31 * rcp_n);
}
__host__ __device__ __forceinline__ uint64_t fix32_at(uint32_t k, uint32_t slope, bool neg, uint32_t start) {
    return (uint64_t)k * slope + (neg && slope != kFix32Always ? start : 0x80000000u);
}
// From a remainder, in float (pieces, N <= 16384, chunks of 32 samples): scale is
// 2^32 times a reciprocal of 2N within one ulp; biased upwards by 2048 units, more
// than the error of less than 1024, so at most 3072 units too large each, below
// 32 x 3072 < 2^32 / 2N after a chunk's 31 steps.
__host__ __device__ __forceinline__ uint32_t fix32_about(uint32_t x, float scale) {
    return (uint32_t)((float)x * scale) + 2048u;
}

// int16 coordinates of eq. (3) in 16.16 fixed point, for N <= kFix16MaxN: the
// high half of P + k d / N, P = p0 + 1/2, is the voxel's coordinate
// p0 + floor((2 k d + N) / 2N) as long as the sum is never below its value and
// less than 1 / 2N above it (values are multiples of 1 / 2N).  fix30_slope is
// d / N in 2^-30, at most 1 + 2^-8 units too large; fix16_at the sum at any
// k <= N, at most N (1 + 2^-8) 2^-14 + 1 < 1.24 units of 2^-16 too large; and
// steps from there add fix16_step, at most 1.001 units too large each.  Seven
// steps stay below 8.3 units, 2^16 / 2N is at least 8.4.
constexpr uint32_t kFix16MaxN = 3900;
__host__ __device__ __forceinline__ int32_t fix30_slope(int32_t d, double rcp_n) {
    return (int32_t)__builtin_ceil((double)d * 0x1p30 * rcp_n + 0x1p-8);
}
__host__ __device__ __forceinline__ int32_t fix16_point(int32_t p0) {
    return (int32_t)(((uint32_t)p0 << 16) + 0x8000u);
}
__host__ __device__ __forceinline__ int32_t fix16_at(int32_t point, int32_t slope, uint32_t k) {
    return (int32_t)((uint32_t)point + (uint32_t)(((int64_t)(int32_t)k * slope + 16383) >> 14));
}
__host__ __device__ __forceinline__ int32_t fix16_step(int32_t slope) { return (slope + 16383) >> 14; }

struct AxisStep {
    uint32_t q, r, two_a;
};

// Quotients and remainders of (2 k a + N - neg) / 2N, per axis, for N >= 1
// and k <= N.  Up to N = 32767 the numerators stay below 2^31 and the
// quotients at most a < 2^15, so one reciprocal serves all three axes
// (divmod_down); beyond that, 64-bit divisions.
__device__ __forceinline__ void axis_init3(const uint32_t a[3], const uint32_t neg[3], uint32_t N, uint32_t k,
                                           AxisStep st[3]) {
    const uint32_t two_n = 2u * N;
    if (N <= 32767u) {
        const float rcpd = rcp_down(two_n);
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            st[ax].two_a = 2u * a[ax];
            divmod_down(2u * k * a[ax] + N - neg[ax], two_n, rcpd, st[ax].q, st[ax].r);
        }
    } else {
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            st[ax].two_a = 2u * a[ax];
            const uint64_t num = 2ull * k * a[ax] + N - neg[ax];
            const uint64_t q = num / two_n;
            st[ax].q = (uint32_t)q;
            st[ax].r = (uint32_t)(num - q * two_n);
        }
    }
}

__device__ __forceinline__ void axis_step(AxisStep& st, uint32_t two_n) {
    st.r += st.two_a;
    bool c = st.r >= two_n;
    st.r = c ? st.r - two_n : st.r;
    st.q += c ? 1u : 0u;
}

// Lanes per segment where a wave takes several segments at once, one sample
// per lane (a power of two dividing 64).
constexpr int kSampleLanes = 16;

// The samples of one segment as taken by one of its kSampleLanes lanes:
// samples k, k + kSampleLanes, k + 2 kSampleLanes, ...  q_a and r_a are the
// quotient and remainder of (2 k a + N - neg) / 2N.  Because a <= N, the
// step from k - 1 to k moves axis a (by one) exactly when it carries, that is
// when r_a(k) < 2a, so a lane knows on its own whether its sample starts a
// new voxel.  start() divides once (one reciprocal for all three axes up to
// N = 32767, where the numerators stay below 2^31 and the quotients below
// 2^15; 64-bit divisions beyond); next() moves on by kSampleLanes samples
// with the per-segment stride (dq, dr) = divmod(kSampleLanes * 2a, 2N), one
// add and one correction per axis.  Both return whether the sample moved
// (true at k = 0).  Samples past N get meaningless values.
struct SampleAt {
    uint32_t two_a[3], num0[3], dq[3], dr[3];
    uint32_t q[3], r[3];
    bool neg[3];
    uint32_t N, two_n;

    __device__ __forceinline__ void init(const Seg& g, uint32_t n) {
        N = n;
        two_n = 2u * n;
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            const int32_t d = g.p1[ax] - g.p0[ax];
            neg[ax] = d < 0;
            two_a[ax] = 2u * (uint32_t)(d < 0 ? -d : d);
            num0[ax] = n - (neg[ax] ? 1u : 0u);
        }
    }

    __device__ __forceinline__ bool start(uint32_t k) {
        bool moved = k == 0;
        if (N == 0) {
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) q[ax] = r[ax] = dq[ax] = dr[ax] = 0;
        } else if (N <= 32767u) {
            const float rcpd = rcp_down(two_n);
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                divmod_down(__umul24(k, two_a[ax]) + num0[ax], two_n, rcpd, q[ax], r[ax]);
                divmod_down(kSampleLanes * two_a[ax], two_n, rcpd, dq[ax], dr[ax]);
                moved |= r[ax] < two_a[ax];
            }
        } else {
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                const uint64_t num = (uint64_t)k * two_a[ax] + num0[ax];
                q[ax] = (uint32_t)(num / two_n);
                r[ax] = (uint32_t)(num - (uint64_t)q[ax] * two_n);
                const uint32_t s = kSampleLanes * two_a[ax];
                dq[ax] = s / two_n;
                dr[ax] = s - dq[ax] * two_n;
                moved |= r[ax] < two_a[ax];
            }
        }
        return moved;
    }

    __device__ __forceinline__ bool next() {
        bool moved = false;
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            const uint32_t t = r[ax] + dr[ax];
            const bool c = t >= two_n;
            r[ax] = c ? t - two_n : t;
            q[ax] += dq[ax] + (c ? 1u : 0u);
            moved |= r[ax] < two_a[ax];
        }
        return moved;
    }

    __device__ __forceinline__ int32_t coord(const Seg& g, int ax) const {
        return g.p0[ax] + (neg[ax] ? -(int32_t)q[ax] : (int32_t)q[ax]);
    }
};

// ------------------------------------------------------------ block scans

template <typename T>
__device__ __forceinline__ T wave_inclusive_sum(T v) {
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        T t = __shfl_up(v, o, kWave);
        if (lane >= o) v += t;
    }
    return v;
}

// Inclusive sum over the 64 lanes of a wave with DPP moves (rows of 16:
// shifts by 1, 2, 4, 8; then row 15 broadcast into rows 1 and 3, lane 31
// into rows 2 and 3).  All lanes must be active.
__device__ __forceinline__ uint32_t wave_inclusive_sum_dpp(uint32_t x) {
    uint32_t s = x;
    s += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)s, 0x111, 0xf, 0xf, true);  // row_shr:1
    s += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)s, 0x112, 0xf, 0xf, true);  // row_shr:2
    s += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)s, 0x114, 0xf, 0xf, true);  // row_shr:4
    s += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)s, 0x118, 0xf, 0xf, true);  // row_shr:8
    s += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)s, 0x142, 0xa, 0xf, false); // row_bcast:15
    s += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)s, 0x143, 0xc, 0xf, false); // row_bcast:31
    return s;
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}

// Exclusive prefix sum over the block (one value per thread, thread order).
// `lds` needs kBlock/64 entries; returns the block total in `total`.
template <int kBlock, typename T>
__device__ __forceinline__ T block_exclusive_sum(T v, T* lds, T& total) {
    constexpr int kWaves = kBlock / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    const int w = threadIdx.x / kWave;
    T incl = wave_inclusive_sum(v);
    if (lane == kWave - 1) lds[w] = incl;
    __syncthreads();
    T pre = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < kWaves; ++i) {
        T x = lds[i];
        pre += (i < w) ? x : T(0);
        tot += x;
    }
    __syncthreads();
    total = tot;
    return pre + incl - v;
}

template <int kBlock, typename T>
__device__ __forceinline__ T block_sum(T v, T* lds) {
    constexpr int kWaves = kBlock / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    const int w = threadIdx.x / kWave;
    v = wave_sum(v);
    if (lane == 0) lds[w] = v;
    __syncthreads();
    T tot = 0;
#pragma unroll
    for (int i = 0; i < kWaves; ++i) tot += lds[i];
    __syncthreads();
    return tot;
}

}  // namespace vox
