// fp32 assignment on the matrix cores, with the answer of the direct fp32 differences.
//
// Direct differences cost two vector instructions per (point, centroid, feature) and leave the
// matrix cores idle.  Here a first kernel only NARROWS the choice: it computes, for every pair,
//     s_k = x'.c'_k - |c'_k|^2 / 2          x' = x - m,  c' = c - m
// (the argmin of |x - c_k|^2 is the argmax of s_k; m, the mean of some of the centroids or points, keeps
// the numbers as small as the data's spread) with x' and c' each split into two bf16 values,
//     x'.c' ~ xh.ch + xl.ch + xh.cl,
// and keeps the best and the second best score of every point.  Where the two are further apart
// than everything that rounding can have done to them -- here and in the direct form -- the best
// one is the one the direct form finds.  The other points go on a list, and a second kernel
// measures them against all centroids by direct differences, with the arithmetic of the
// stand-alone kernels (fk_assign.hip).  The assignments are therefore those of the direct
// kernels bit for bit, ties and all, whatever the data; only the time depends on it.
//
// What rounding can do, with S_k = |x'|^2 + |c'_k|^2 and D = padded row width (|x||c| <= S/2):
//   xl.cl and the two remainders of the splits           <= 3 2^-18 |x||c|      <= 1.5 2^-18 S
//   every one of the D + 16 additions of the chain xh.ch + bias, at most 2^-23 of a partial sum
//   that is at most |x||c| (1 + 2^-7), plus |c|^2/2 in the last 16  <= (0.51 D + 20) 2^-23 S
//   (measured: 16 of them, one MFMA, are off by at most 1.8 2^-23 of the sum of the magnitudes of
//   their terms, and 7.5 2^-23 of the largest, over terms up to 2^46 apart, with and without signs)
//   the 2 D additions of the small products, partial sums <= 2^-7 |x||c|       <= 0.01 D 2^-23 S
//   adding the two accumulators, bias to 24 bits, rounding of x - m and c - m  <= 4 2^-23 S
//   the four low bits of a score that carry its slot           <= 15 2^-23 S = 0.94 2^-19 S
// together kappa S with kappa = 2^-17 + (0.53 D + 24) 2^-23 (the first and last lines are below
// 2^-17).  The |c'_k|^2 part of it is added to the score of k through its bias, so the scores
// kept are upper bounds less kappa |x'|^2, and centroid 1 is certain when
//     u_1 - u_2  >  2 kappa (|x'|^2 + |c'_1|^2) + theta,
// where theta covers the direct form's own rounding, (d + 3) 2^-24 of a distance near the best
// one's, |x'|^2 - 2 s_1.  Anything that is not finite fails the test and goes on the list.
//
// What bounds it: the matrix pipe (3 MFMA per 32 points x 32 centroids x 16 features, 6 N K D
// flop) from about 64 centroids up, below that reading X.
#include <algorithm>
#include <type_traits>

#include "fk_common.h"
#include "fk_device.h"

namespace fk {

namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{a, b}, bf16x2));
}

// eight fp32 values -> their bf16 heads and the bf16 roundings of what the heads leave
__device__ __forceinline__ void split8(const float (&v)[8], uintx4& hi, uintx4& lo) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t w = pack_bf16(v[2 * q], v[2 * q + 1]);
        hi[q] = w;
        lo[q] = pack_bf16(v[2 * q] - __uint_as_float(w << 16), v[2 * q + 1] - __uint_as_float(w & 0xFFFF0000u));
    }
}

}  // namespace

// One workgroup per centroid tile (32 rows).  Writes the tile as MFMA A operands, 1 KiB pieces in
// the order  head, tail of chunk 0;  head, tail of chunk 1;  ...;  bias,  where the bias piece
// holds u-bias -|c'|^2/2 + kappa |c'|^2 as three bf16 values (24 bits) in its first features, to
// be multiplied by ones.  A row whose norm overflows gets zeros and a bias that always wins, with
// c2 = inf, so that no point is ever certain of it; rows past K one that never wins.  Rows with a NaN
// or an infinity get that too -- no distance to them is below infinity, where the direct form's minimum
// starts -- and stay out of the mean: one such centroid would leave every point open.
// The mean of up to 32 of the centroids or, where X is given (fits, whose later iterations keep the shift, see emit_split in
// fk_update.hip), of half of 32 of the points (point_mean): the centroids that a fit starts from may lie anywhere, the
// later ones lie among the points.
// Tile 0 also leaves the shift m and clears the lengths of the instance's lists.
// A few microseconds of dependent loads, and of instructions that no cache holds yet: the rows of the mean are asked for eight at a
// time and the own rows before the mean is needed, and nothing is in the code that the shape has no use for (kGroups, RAGGED; d = 128, K = 211
// 7.2 -> 5.5 us; with all 32 rows of the mean asked for at once 7.6).
constexpr int kLayoutThreads = 512;

// Feature x of 32 of N rows (sampled_row).  Of four means of eight the largest and the smallest stay out, and with them a row far off.
// (64 rows: a fit of 300000 points, d = 96, K = 400 takes 2 us more.)
__device__ __forceinline__ float point_mean(const float* __restrict__ x, uint32_t N, int len) {
    float a = 0.f, b = 0.f, c = 0.f, e = 0.f;
#pragma unroll 1
    for (uint32_t i0 = 0; i0 < 32; i0 += 8) {
        float v[8], s = 0.f;
#pragma unroll
        for (uint32_t i = 0; i < 8; ++i) v[i] = x[(size_t)sampled_row(i0 + i, N) * len];
#pragma unroll
        for (int i = 0; i < 8; ++i) s += fabsf(v[i]) < INFINITY ? v[i] * 0.125f : 0.f;
        a = b; b = c; c = e; e = s;
    }
    return 0.5f * (fmaxf(fminf(a, b), fminf(c, e)) + fminf(fmaxf(a, b), fmaxf(c, e)));
}

template <int kGroups, bool RAGGED>
__global__ __launch_bounds__(kLayoutThreads) void f32_split_layout_kernel(
    const float* __restrict__ X, uint32_t N, const float* __restrict__ C, uintx4* __restrict__ frag, float* __restrict__ c2,
    float* __restrict__ shift, int32_t* __restrict__ list_len, int32_t* __restrict__ pair_len, int d, int row_len, int K, int ktiles, int dch) {
    const int len = RAGGED ? row_len : d;
    __shared__ float m[512];
    __shared__ double part[32][65];
    __shared__ int fits[32], odd_row[32];
    const int b = blockIdx.y, kt = blockIdx.x, tid = threadIdx.x;
    const int width = dch * 16;
    C += (size_t)b * K * len;
    frag += ((size_t)b * ktiles + kt) * (2 * dch + 1) * 64;
    // this thread's groups of eight features: group g = tid + i * threads is lane g % 64 of chunk g / 64
    float own[kGroups][8];
#pragma unroll
    for (int i = 0; i < kGroups; ++i) {
        const int g = tid + i * kLayoutThreads;
        const int l = g & 63, k = kt * 32 + (l & 31), j0 = (g >> 6) * 16 + (l >> 5) * 8;
#pragma unroll
        for (int e = 0; e < 8; ++e) own[i][e] = 0.f;
        if (g < 64 * dch && k < K && j0 < d) {
            const floatx4 u = row_piece32<RAGGED>(C + (size_t)k * len, j0, len), v = row_piece32<RAGGED>(C + (size_t)k * len, j0 + 4, len);
#pragma unroll
            for (int e = 0; e < 4; ++e) { own[i][e] = u[e]; own[i][e + 4] = v[e]; }
        }
    }
    const int rows = min(K, 32);
    if (tid < width) {
        float s = 0.f;
        if (tid < len && X) {
            s = point_mean(X + (size_t)b * N * len + tid, N, len);
        } else if (tid < len) {
#pragma unroll 1
            for (int i0 = 0; i0 < rows; i0 += 8) {
                float v[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = C[(uint32_t)min(i0 + i, rows - 1) * (uint32_t)K / (uint32_t)rows * (uint32_t)len + tid];
#pragma unroll
                for (int i = 0; i < 8; ++i) s += i0 + i < rows && fabsf(v[i]) < INFINITY ? v[i] : 0.f;
            }
            s /= (float)rows;
        }
        m[tid] = s;
        if (kt == 0) shift[(size_t)b * width + tid] = s;
    }
    if (tid < 32) odd_row[tid] = 0;
    if (kt == 0 && tid == 0) { list_len[b] = 0; pair_len[b] = 0; }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kGroups; ++i) {
        const int g = tid + i * kLayoutThreads;
        const int l = g & 63, k = kt * 32 + (l & 31), j0 = (g >> 6) * 16 + (l >> 5) * 8;
        if (g < 64 * dch) {
            double ss = 0.0;
            bool odd = false;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                odd |= !(fabsf(own[i][e]) < INFINITY);
                own[i][e] = k < K && j0 < d ? own[i][e] - m[j0 + e] : 0.f;
                ss += (double)own[i][e] * (double)own[i][e];
            }
            part[l & 31][(g >> 6) * 2 + (l >> 5)] = ss;
            if (odd) odd_row[l & 31] = 1;
        }
    }
    __syncthreads();
    {
        // sixteen lanes a row
        const int r = tid >> 4, c = tid & 15, k = kt * 32 + r;
        double n2 = 0.0;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (c + 16 * q < 2 * dch) n2 += part[r][c + 16 * q];
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) n2 += __shfl_xor(n2, o);
        if (c < 2) {
            const bool never = k >= K || odd_row[r] != 0;
            float norm;
            uintx4 v = split_bias(n2, width, never, &norm);
            if (c == 0) {
                fits[r] = !never && n2 < 1e38;
                c2[((size_t)b * ktiles + kt) * 32 + r] = norm;
            } else {
                v = uintx4{0u, 0u, 0u, 0u};
            }
            frag[2 * dch * 64 + c * 32 + r] = v;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kGroups; ++i) {
        const int g = tid + i * kLayoutThreads;
        if (g < 64 * dch) {
            const int l = g & 63, s = g >> 6;
            if (!fits[l & 31])
#pragma unroll
                for (int e = 0; e < 8; ++e) own[i][e] = 0.f;
            uintx4 hi, lo;
            split8(own[i], hi, lo);
            frag[(2 * s) * 64 + l] = hi;
            frag[(2 * s + 1) * 64 + l] = lo;
        }
    }
}

// What a lane keeps of its scores: the best and the second best (low 4 bits = 15 - slot) with their tiles and, where
// THREE, the value of the third, so that a point that is open between two centroids only need not be measured against
// all of them.
// (Rows of more than 96 features: narrower ones are measured in full sooner than the sweep takes one more operation a score, 300000
// points, d = 96, K = 400 399 us a fit for 386, 598071, d = 32, K = 75 312 for 287.)
constexpr bool filter_keeps_three(int dch) { return dch >= 7; }

template <bool THREE>
struct TopScores {
    float m1, m2, m3;
    int t1, t2;                                              // tiles; after settle(): centroids

    __device__ __forceinline__ void clear() { m1 = m2 = m3 = -INFINITY; t1 = t2 = 0; }
    __device__ __forceinline__ void fold(const floatx16& big, const floatx16& small, int tile) {
        const float before1 = m1, before2 = m2;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const float u = __uint_as_float((__float_as_uint(big[i] + small[i]) & 0xFFFFFFF0u) | (uint32_t)(15 - i));
            if constexpr (THREE) m3 = __builtin_amdgcn_fmed3f(m2, m3, u);
            m2 = __builtin_amdgcn_fmed3f(m1, m2, u);
            m1 = __builtin_fmaxf(m1, u);
        }
        // (equal scores may be given the wrong tile: the third is then as good as the second, and the point measured in full)
        if constexpr (THREE) t2 = m2 == before2 ? t2 : m2 == before1 && m1 != before1 ? t1 : tile;
        t1 = m1 != before1 ? tile : t1;
    }
    __device__ __forceinline__ static int centroid(float m, int tile, int h) {
        const int i = 15 - (int)(__float_as_uint(m) & 15u);
        return tile * 32 + 8 * (i >> 2) + 4 * h + (i & 3);
    }
    __device__ __forceinline__ void settle(int h) {
        t1 = centroid(m1, t1, h);
        if constexpr (THREE) t2 = centroid(m2, t2, h);
    }
    __device__ __forceinline__ void merge(const TopScores& o) {
        if constexpr (THREE) m3 = __builtin_fmaxf(__builtin_fmaxf(m3, o.m3), __builtin_fmaxf(__builtin_fminf(m1, o.m2), __builtin_fminf(m2, o.m1)));
        const bool other = o.m1 > m1;
        const float low = other ? m1 : o.m1, next = other ? o.m2 : m2;
        if constexpr (THREE) {
            const int low_k = other ? t1 : o.t1, next_k = other ? o.t2 : t2;
            t2 = low > next ? low_k : next_k;
        }
        m2 = __builtin_fmaxf(low, next);
        t1 = other ? o.t1 : t1;
        m1 = other ? o.m1 : m1;
    }
    __device__ __forceinline__ void merge_halves(int h) {    // the two lanes of a point meet
        settle(h);
        TopScores o;
        o.clear();
        o.m1 = __shfl_xor(m1, 32);
        o.m2 = __shfl_xor(m2, 32);
        o.t1 = __shfl_xor(t1, 32);
        if constexpr (THREE) {
            o.m3 = __shfl_xor(m3, 32);
            o.t2 = __shfl_xor(t2, 32);
        }
        merge(o);
    }
    // 0: t1 it is; 1: t1 or t2; 2: open.  x2 = |x'|^2, c2 = |c'|^2 by centroid.
    __device__ __forceinline__ int verdict(float x2, const float* __restrict__ c2, int width, int d, int K) {
        t1 = min(t1, K - 1);
        const float room = 2.02f * filter_kappa(width) * (x2 + c2[t1]);
        // distance to the best one, from above (u_1 is s_1 + kappa |c'_1|^2 give or take room / 2)
        const float near = fmaxf(0.f, x2 - 2.f * m1) + 3.f * room;
        const float theta = (float)(d + 4) * 5.9604645e-08f * 1.1f * near;
        if (m1 - m2 > room + theta + 1e-30f) return 0;
        return THREE && m1 - m3 > room + theta + 1e-30f ? 1 : 2;
    }
};

// Open points carry -1 where distances are wanted, whose place then holds the two centroids (see assign_f32_list_kernel).
__device__ __forceinline__ void leave_verdict(int k1, int k2, int verdict, bool mine, int64_t point, int K, int32_t* __restrict__ assign,
                                              int32_t* __restrict__ pair_at) {
    if (!mine) return;
    const int32_t both = (int32_t)((uint32_t)k1 | ((uint32_t)min(k2, K - 1) << 16));
    if (pair_at && verdict == 1) pair_at[point] = both;
    if (verdict == 0 || verdict == 1 || pair_at) assign[point] = verdict == 0 ? k1 : pair_at ? -1 : both;
}

// The sweep.  As in the 16-bit kernels a wave owns 32 points, whose features stay in registers as
// B operands (heads and tails: 8 DCH registers per lane), and the centroid tiles pass through a
// double-buffered LDS stage of eight chunks that is filled by direct copies; a lane holds 16
// centroid rows of one point.  The head product and the two small products have accumulators of
// their own, which keeps the rounding of the small ones small and gives two independent chains.
// Waves per SIMD that the registers are held to: what the kernel has without reading ahead (none of these spills).
constexpr int filter_occupancy(int dch, int waves) {
    return waves == 8 || dch <= 3 || dch == 7 || dch == 12 ? 1 : dch <= 6 ? 4 : dch <= 10 ? 3 : dch <= 16 ? 2 : 1;
}

template <int DCH, int WAVES>
__global__ __launch_bounds__(WAVES * 64, filter_occupancy(DCH, WAVES)) void assign_f32_filter_kernel(
    const float* __restrict__ X, const uintx4* __restrict__ frag, const float* __restrict__ c2,
    const float* __restrict__ shift, int32_t* __restrict__ assign, int32_t* __restrict__ list,
    int32_t* __restrict__ list_len, int32_t* __restrict__ pair_len, int32_t* __restrict__ pair_at, int64_t N, int d, int len, int K, int ktiles) {
    constexpr int kTile = 2 * DCH + 1;                       // 1 KiB pieces per centroid tile
    constexpr int ST = DCH < 8 ? 8 / DCH : 1;                // tiles per stage ...
    constexpr int SPT = DCH <= 8 ? 1 : DCH <= 16 ? 2 : 4;    // ... or stages per tile
    constexpr int SC = DCH / SPT;                            // chunks of a tile in one stage
    constexpr int kPieces = SPT > 1 ? 2 * SC + 1 : ST * kTile;   // pieces per stage, at most
    static_assert(SC * SPT == DCH, "whole chunks per stage");
    // Four waves: two objects, and code for each, since with one array every operand read waits for the copy in
    // flight into the other half; and the operands of a chunk are read while the one before is multiplied (a wave alone on
    // its SIMD otherwise waits as long for LDS as it multiplies).  Sweep, us, medians of 300 launches: 50000 points, d = 512,
    // K = 1000 251 -> 227; 5000, d = 333, K = 5000 393 -> 335; 300000, d = 96, K = 400 99.3 -> 97.8; 1317, d = 512, K = 293
    // 43.9 -> 39.7.  Eight waves have no registers left for either (2^20 points, d = 128, K = 64 127 us, 162 with two objects,
    // 180 with both), nor have three chunks at their five waves a SIMD (58.1, 59.0), seven at four (93, 108) and twelve at three:
    // with 12 registers spilled fk_assign of 8000 points, d = 192, K = 2000 91.5 -> 96.7, 600000, K = 200 204 -> 213; with two waves
    // 87.5 and 216.  Twelve chunks as they were need the order of reads and products kept (92.0 and 204; 96.7 without).
    constexpr bool kApart = WAVES == 4 && DCH != 3 && DCH != 7 && DCH != 12;
    constexpr bool kInTurn = kApart || SPT > 1;
    __shared__ uintx4 even[(kApart ? 1 : 2) * kPieces * 64], other_half[kApart ? kPieces * 64 : 1];
    uintx4* const odd = kApart ? other_half : even + kPieces * 64;

    const int b = blockIdx.y;
    X += (size_t)b * N * len;
    frag += (size_t)b * ktiles * kTile * 64;
    c2 += (size_t)b * ktiles * 32;
    shift += (size_t)b * DCH * 16;
    assign += (size_t)b * N;
    list += (size_t)b * N;
    if (pair_at) pair_at += (size_t)b * N;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = lane & 31, h = lane >> 5;
    const int64_t point = ((int64_t)blockIdx.x * WAVES + wave) * 32 + n;
    const int nst = SPT > 1 ? ktiles * SPT : (ktiles + ST - 1) / ST;

    auto fetch = [&](int st, uintx4* to) {
        const int first = SPT > 1 ? (st / SPT) * kTile + (st % SPT) * 2 * SC : st * kPieces;
        const int count = SPT > 1 ? (st % SPT == SPT - 1 ? 2 * SC + 1 : 2 * SC) : min(kPieces, ktiles * kTile - first);
#pragma unroll
        for (int q = 0; q < (kPieces + WAVES - 1) / WAVES; ++q) {
            const int pc = q * WAVES + wave;                 // wave-uniform
            if (pc < count)
                __builtin_amdgcn_global_load_lds(
                    (const __attribute__((address_space(1))) void*)(frag + (size_t)(first + pc) * 64 + lane),
                    (__attribute__((address_space(3))) void*)(to + pc * 64), 16, 0, 0);
        }
    };
    fetch(0, even);

    uintx4 xh[DCH], xl[DCH];
    float x2 = 0.f;
    auto take = [&](int s, floatx4 a, floatx4 c) {           // features [16 s + 8 h, + 8) of the point
        const int j0 = s * 16 + h * 8;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = 0.f;
        if (point < N && j0 < d) {
            const floatx4 ma = *(const floatx4*)(shift + j0), mc = *(const floatx4*)(shift + j0 + 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] = a[e] - ma[e];
                v[e + 4] = c[e] - mc[e];
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) x2 = fmaf(v[e], v[e], x2);
        }
        split8(v, xh[s], xl[s]);
    };
    const float* row = X + (size_t)(point < N ? point : 0) * len;
    if (len == d) {
#pragma unroll
        for (int s = 0; s < DCH; ++s) {
            const int j0 = min(s * 16 + h * 8, d - 8);
            take(s, *(const floatx4*)(row + j0), *(const floatx4*)(row + j0 + 4));
        }
    } else {
        constexpr int kAhead = DCH % 4 == 0 ? 4 : DCH % 3 == 0 ? 3 : DCH % 5 == 0 ? 5 : DCH % 2 == 0 ? 2 : 1;
#pragma unroll
        for (int s0 = 0; s0 < DCH; s0 += kAhead) {           // a few chunks' loads at a time, then settle them
            floatx4 a[kAhead], c[kAhead];
#pragma unroll
            for (int q = 0; q < kAhead; ++q) {
                const int j0 = min((s0 + q) * 16 + h * 8, d - 8);
                a[q] = raw_piece32(row, j0, len);
                c[q] = raw_piece32(row, j0 + 4, len);
            }
#pragma unroll
            for (int q = 0; q < kAhead; ++q) {
                const int j0 = min((s0 + q) * 16 + h * 8, d - 8);
                take(s0 + q, settle32(a[q], j0, len), settle32(c[q], j0 + 4, len));
            }
        }
    }
    // the ones that the bias piece is multiplied by
    const uintx4 ones = {h == 0 ? 0x3F803F80u : 0u, h == 0 ? 0x3F80u : 0u, 0u, 0u};

    constexpr bool kThree = filter_keeps_three(DCH);
    TopScores<kThree> top;
    top.clear();
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    floatx16 big, small;
    // `chunks` chunks from `at` on, which are the point's from s0 on
    auto products = [&](const uintx4* at, int s0, auto chunks) {
        constexpr int kChunks = decltype(chunks)::value;
        uintx4 ah, al, nh = at[lane], nl = at[64 + lane];
        if constexpr (kInTurn) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);         // two LDS reads
#pragma unroll
        for (int s = 0; s < kChunks; ++s) {
            if (kApart || s == 0) { ah = nh; al = nl; }
            if (kApart && s + 1 < kChunks) {
                nh = at[(2 * s + 2) * 64 + lane];
                nl = at[(2 * s + 3) * 64 + lane];
                __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            } else if (!kApart && s > 0) {
                ah = at[2 * s * 64 + lane];
                al = at[(2 * s + 1) * 64 + lane];
                if constexpr (kInTurn) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            }
            small = mfma32<true>(ah, xl[s0 + s], small);
            big = mfma32<true>(ah, xh[s0 + s], big);
            small = mfma32<true>(al, xh[s0 + s], small);
            if constexpr (kInTurn) __builtin_amdgcn_sched_group_barrier(0x8, 3, 0);       // three MFMAs
        }
    };
    auto fold = [&](const uintx4* bias, int tile) {
        big = mfma32<true>(bias[lane], ones, big);
        top.fold(big, small, tile);
    };
    // stage st, whose pieces are in `now`; the next one's land in `then` meanwhile
    auto sweep = [&](int st, int part, const uintx4* now, uintx4* then) {
        if (st + 1 < nst) fetch(st + 1, then);
        if constexpr (SPT > 1) {
            if (part == 0) { big = floatx16{}; small = floatx16{}; }
            products(now, part * SC, std::integral_constant<int, SC>());
            if (part == SPT - 1) fold(now + 2 * SC * 64, st / SPT);
        } else {
            const int nt = min(ST, ktiles - st * ST);
            for (int tt = 0; tt < nt; ++tt) {
                const uintx4* tile = now + tt * kTile * 64;
                big = floatx16{};
                small = floatx16{};
                products(tile, 0, std::integral_constant<int, DCH>());
                fold(tile + 2 * DCH * 64, st * ST + tt);
            }
        }
        if (st + 1 < nst) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    };
    if constexpr (kApart) {
        static_assert(SPT == 1 || SPT % 2 == 0, "a tile starts in `even`");
        constexpr int kStep = SPT > 1 ? SPT : 2;
        for (int st0 = 0; st0 < nst; st0 += kStep) {
#pragma unroll
            for (int i = 0; i < kStep; i += 2) {
                sweep(st0 + i, i, even, odd);
                if (SPT > 1 || st0 + i + 1 < nst) sweep(st0 + i + 1, i + 1, odd, even);
            }
        }
    } else {
        for (int st0 = 0; st0 < nst; st0 += SPT) {
#pragma unroll
            for (int part = 0; part < SPT; ++part) {
                const int half = (SPT > 1 ? part : st0) & 1;
                sweep(st0 + part, part, even + half * kPieces * 64, even + (half ^ 1) * kPieces * 64);
            }
        }
    }

    top.merge_halves(h);
    x2 += __shfl_xor(x2, 32);
    const int verdict = top.verdict(x2, c2, DCH * 16, d, K);
    const bool mine = h == 0 && point < N;
    leave_verdict(top.t1, top.t2, verdict, mine, point, K, assign, pair_at);
    // A place on the list for the whole workgroup at once: additions to one address take 10 ns each, and
    // with many open points one per wave cost more than the sweep (2^20 points, all open: 330 us).
    // (The last stage has been read; LDS of its own would cost a workgroup per compute unit at DCH = 2.)
    // Open points go on the list from its front, those open between two centroids from its end.
    int* opened = (int*)&even[0];
    int* list_at = opened + 2 * WAVES;
    const uint64_t below = (1ull << lane) - 1ull;
    const uint64_t open = __ballot(mine && verdict == 2), pair = kThree ? __ballot(mine && verdict == 1) : 0;
    if (lane == 0) {
        opened[wave] = __popcll(open);
        if constexpr (kThree) opened[WAVES + wave] = __popcll(pair);
    }
    __syncthreads();
    int before = 0, all = 0, pairs_before = 0, pairs = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        const int c = opened[w];
        before += w < wave ? c : 0;
        all += c;
        if constexpr (kThree) {
            const int p = opened[WAVES + w];
            pairs_before += w < wave ? p : 0;
            pairs += p;
        }
    }
    if (all + pairs == 0) return;
    if (tid == 0 && all > 0) list_at[0] = atomicAdd(list_len + b, all);
    if (kThree && tid == 1 && pairs > 0) list_at[1] = atomicAdd(pair_len + b, pairs);
    __syncthreads();
    if (mine && verdict == 2) list[list_at[0] + before + __popcll(open & below)] = (int32_t)point;
    if (kThree && mine && verdict == 1) list[N - 1 - (list_at[1] + pairs_before + __popcll(pair & below))] = (int32_t)point;
}

// Few points: a workgroup of the sweep has 128 and walks through all centroids alone, so that a few thousand points keep
// a few compute units busy.  Here it has 32, its waves share out the centroid tiles, and nothing but the points and the waves' best scores
// passes through LDS: the operands of a tile come straight from memory (from L2, where all workgroups find them), half a tile or less
// ahead of their use.  Same scores, same verdicts.  fk_assign, us, in the sweep / here: 2415 points, d = 128, K = 3561 116 / 37; 2 x 5764,
// d = 415, K = 767 138 / 103; 8000, d = 512, K = 4000 551 / 309; an iteration of 2 x 3027, d = 242, K = 609 69 / 47.
constexpr int few_ahead(int dch) { return dch % 4 == 0 ? 4 : dch % 3 == 0 ? 3 : dch % 5 == 0 ? 5 : dch % 7 == 0 ? 7 : dch % 2 == 0 ? 2 : 1; }
constexpr int kFewWaves = 8;

template <int DCH>
__global__ __launch_bounds__(kFewWaves * 64, DCH <= 3 ? 4 : 2) void assign_f32_filter_few_kernel(
    const float* __restrict__ X, const uintx4* __restrict__ frag, const float* __restrict__ c2,
    const float* __restrict__ shift, int32_t* __restrict__ assign, int32_t* __restrict__ list,
    int32_t* __restrict__ list_len, int32_t* __restrict__ pair_len, int32_t* __restrict__ pair_at, int64_t N, int d, int len, int K, int ktiles) {
    constexpr int WAVES = kFewWaves, kTile = 2 * DCH + 1, GC = few_ahead(DCH), NG = DCH / GC;
    constexpr bool kThree = filter_keeps_three(DCH);
    constexpr bool kHeld = DCH <= 16 && DCH != 14;           // the points' operands stay in registers (14: they would spill)
    // heads and tails of the 32 points, as B operands; at the end the waves' best scores
    __shared__ uintx4 xs[2 * DCH * 64 > WAVES * 40 ? 2 * DCH * 64 : WAVES * 40];
    __shared__ float sums[WAVES][32];
    auto found = (TopScores<kThree>(*)[32])xs;
    static_assert(sizeof(found[0]) * WAVES <= sizeof(xs), "room for the best scores");
    const int b = blockIdx.y;
    X += (size_t)b * N * len;
    frag += (size_t)b * ktiles * kTile * 64;
    c2 += (size_t)b * ktiles * 32;
    shift += (size_t)b * DCH * 16;
    assign += (size_t)b * N;
    list += (size_t)b * N;
    if (pair_at) pair_at += (size_t)b * N;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = lane & 31, h = lane >> 5;
    const int64_t point = (int64_t)blockIdx.x * 32 + n;

    // step: group of GC chunks of one of this wave's tiles
    const int tiles = wave < ktiles ? (ktiles - wave + WAVES - 1) / WAVES : 0;
    uintx4 ahead[2 * GC];
    auto load = [&](int t, int g) {
        const uintx4* at = frag + ((size_t)(wave + t * WAVES) * kTile + 2 * g * GC) * 64 + lane;
#pragma unroll
        for (int q = 0; q < 2 * GC; ++q) ahead[q] = at[q * 64];
    };
    if (tiles > 0) load(0, 0);
    float x2 = 0.f;
    const float* row = X + (size_t)min(point, N - 1) * len;
    for (int s = wave; s < DCH; s += WAVES) {
        const int j0 = s * 16 + h * 8;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = 0.f;
        if (point < N && j0 < d) {
            const floatx4 a = row_piece32(row, j0, len), c = row_piece32(row, j0 + 4, len);
            const floatx4 ma = *(const floatx4*)(shift + j0), mc = *(const floatx4*)(shift + j0 + 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) { v[e] = a[e] - ma[e]; v[e + 4] = c[e] - mc[e]; }
#pragma unroll
            for (int e = 0; e < 8; ++e) x2 = fmaf(v[e], v[e], x2);
        }
        uintx4 hi, lo;
        split8(v, hi, lo);
        xs[2 * s * 64 + lane] = hi;
        xs[(2 * s + 1) * 64 + lane] = lo;
    }
    x2 += __shfl_xor(x2, 32);
    if (h == 0) sums[wave][n] = x2;
    __syncthreads();
    uintx4 xh[kHeld ? DCH : 1], xl[kHeld ? DCH : 1];
    if constexpr (kHeld) {
#pragma unroll
        for (int s = 0; s < DCH; ++s) { xh[s] = xs[2 * s * 64 + lane]; xl[s] = xs[(2 * s + 1) * 64 + lane]; }
    }
    const uintx4 ones = {h == 0 ? 0x3F803F80u : 0u, h == 0 ? 0x3F80u : 0u, 0u, 0u};
    TopScores<kThree> top;
    top.clear();
    for (int t = 0; t < tiles; ++t) {
        const int tile = wave + t * WAVES;
        const uintx4 bias = frag[((size_t)tile * kTile + 2 * DCH) * 64 + lane];
        floatx16 big = floatx16{}, small = floatx16{};
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            uintx4 now[2 * GC];
#pragma unroll
            for (int q = 0; q < 2 * GC; ++q) now[q] = ahead[q];
            if (!kHeld) asm volatile("" ::: "memory");    // (or they are all read before the loop)
            if (g + 1 < NG) load(t, g + 1);
            else if (t + 1 < tiles) load(t + 1, 0);
#pragma unroll
            for (int q = 0; q < GC; ++q) {
                const int s = g * GC + q;
                const uintx4 bh = kHeld ? xh[kHeld ? s : 0] : xs[2 * s * 64 + lane], bl = kHeld ? xl[kHeld ? s : 0] : xs[(2 * s + 1) * 64 + lane];
                small = mfma32<true>(now[2 * q], bl, small);
                big = mfma32<true>(now[2 * q], bh, big);
                small = mfma32<true>(now[2 * q + 1], bh, small);
            }
        }
        big = mfma32<true>(bias, ones, big);
        top.fold(big, small, tile);
    }
    top.merge_halves(h);
    __syncthreads();                                         // (the operands have been read)
    if (h == 0) found[wave][n] = top;
    __syncthreads();
    if (wave != 0) return;
    x2 = sums[0][n];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) {
        x2 += sums[w][n];
        if (w < ktiles) top.merge(found[w][n]);
    }
    const int verdict = top.verdict(x2, c2, DCH * 16, d, K);
    const bool mine = h == 0 && point < N;
    leave_verdict(top.t1, top.t2, verdict, mine, point, K, assign, pair_at);
    const uint64_t below = (1ull << lane) - 1ull;
    const uint64_t open = __ballot(mine && verdict == 2), pair = kThree ? __ballot(mine && verdict == 1) : 0;
    int at = 0, pair_from = 0;
    if (lane == 0 && open) at = atomicAdd(list_len + b, __popcll(open));
    if (lane == 0 && pair) pair_from = atomicAdd(pair_len + b, __popcll(pair));
    at = __builtin_amdgcn_readfirstlane(at);
    pair_from = __builtin_amdgcn_readfirstlane(pair_from);
    if (mine && verdict == 2) list[at + __popcll(open & below)] = (int32_t)point;
    if (kThree && mine && verdict == 1) list[N - 1 - (pair_from + __popcll(pair & below))] = (int32_t)point;
}

// The points on the list against all centroids by direct differences: ascending features, one
// fused multiply-add each, ascending centroids with strict '<' -- the same operations in the same
// order as assign_f32_kernel.
//   As a rule lane = centroid row, read 128 bytes at a time, a block of features ahead of its use;
// a wave holds P points.  The eight waves of a workgroup share out the centroids or, where those
// are too few, take points of their own (`teams` of 8 / teams waves each).  With P = 2 a short
// list is spread thin and over in the time that a few rows take to arrive (5 to 20 us); with P =
// 8 a long one is bound by reading its points from LDS, a pass of which serves 64 centroids, so that its waves take points of their
// own as soon as all workgroups have some: waves that share 400 rows leave one of eight idle, 300 three (every centroid twice, 300000 points,
// d = 96, K = 400 1306 -> 890 us, 400000, d = 80, K = 300 1460 -> 710, 20000 94 -> 69).
//   Long lists of rows of up to 64 features, where that form spends its time on reading centroid
// rows: one point per thread with its features in registers, centroid tiles through LDS.  (Not rows of
// up to 16 against many centroids: it multiplies 32 features.  7 x 294694 points, d = 8, K = 14868: 60.1 ms
// against 34.4.)
//   Points that are open between two centroids only, nineteen of twenty where the filter keeps three scores, are on a list of
// their own and cost two rows each (list_pairs).  fk_assign of 65536 points, d = 256, K = 512, distances: 1837 such points and 42 others,
// list and distances 44 -> 22 us.
//   What other open points cost is about the direct kernel's time for them, or less, on top of the filter's.
// All points open, fk_assign against the direct kernels alone, us.  Every centroid twice: 2^20 points,
// d = K = 64: 278, 221 (one addition to the list's length per wave: 610); d = 64, K = 256: 831, 811
// (in the first form: 1896); d = 128, K = 64: 389, 640 (pairs); 300000 points, d = 96, K = 400:
// 874, 1154; 65536, d = 256, K = 512: 89, 1341 (pairs).  Four times: d = 128, K = 64: 871, 640; 65536, d = 256, K = 512: 557, 1348.

// |x - c|^2 by direct differences for every point whose distance is wanted: LANES (4, 8 or 16) lanes a point, enough for a whole
// row per load where it has up to 64 features.  Infinity where it is not finite, as in the direct kernels, whose
// minimum starts there.  (The lanes' sums meet in a butterfly: lanes without a piece add zero, so that their number changes no bit.)
constexpr int distance_lanes(int len) { return len <= 16 ? 4 : len <= 32 ? 8 : 16; }

template <int LANES>
__device__ __forceinline__ float sum_of_lanes(float s) {
#pragma unroll
    for (int o = LANES / 2; o > 0; o >>= 1) s += __shfl_xor(s, o);
    return s < INFINITY ? s : INFINITY;
}

template <int LANES, int U>
__device__ __forceinline__ void row_distances(const float* const (&x)[U], const float* const (&c)[U], int len, int l, float (&s)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) s[u] = 0.f;
    for (int j = l * 4; j < len; j += 4 * LANES) {
        floatx4 v[U], w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) { v[u] = row_piece32(x[u], j, len); w[u] = row_piece32(c[u], j, len); }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) { const float t = v[u][e] - w[u][e]; s[u] = fmaf(t, t, s[u]); }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) s[u] = sum_of_lanes<LANES>(s[u]);
}

// Share `part` of `parts` of the points, by 512 threads, U points at a time a group of lanes; open points (-1) are left out.
// fk_assign with distances, K = 200, us, one / two / four at a time: 400000 points, d = 64 97 / 86 / 81, d = 128 145 / 130 / 125; d = 256,
// 65536, K = 512 84.6 / 85.9 / 86.6, 200000, K = 100 120 / 111 / 111.  The assignment of the next ones is asked for before these are measured,
// and no more than sixteen workgroups a compute unit take turns: 1353626 points, d = 59, K = 26, a workgroup for every 128 points without that
// 213, four / eight / sixteen a unit with it 219 / 205 / 197.
template <int LANES, int U>
__device__ __forceinline__ void measure_points(const float* __restrict__ X, const float* __restrict__ C, const int32_t* assign,
                                               float* min_dist, int64_t N, int len, int64_t part, int64_t parts) {
    constexpr int each = 512 / LANES;
    const int l = threadIdx.x & (LANES - 1);
    int next[U];
    auto ids = [&](int64_t i0) {
#pragma unroll
        for (int u = 0; u < U; ++u) next[u] = __hip_atomic_load(assign + min(i0 + u * each, N - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    ids(part * (U * each) + threadIdx.x / LANES);
    for (int64_t i0 = part * (U * each) + threadIdx.x / LANES; i0 < N; i0 += parts * (U * each)) {
        int k[U];
#pragma unroll
        for (int u = 0; u < U; ++u) k[u] = i0 + u * each < N ? next[u] : -1;
        ids(i0 + parts * (U * each));
        const float *x[U], *c[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            x[u] = X + (size_t)min(i0 + u * each, N - 1) * len;
            c[u] = C + (size_t)max(k[u], 0) * len;
        }
        float s[U];
        row_distances<LANES, U>(x, c, len, l, s);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (l == 0 && k[u] >= 0) min_dist[i0 + u * each] = s[u];
    }
}

// Points held by a workgroup x row width, in floats.  Wide rows: enough that with few centroids as few
// waves as possible are without a share of them.
template <int DMAX>
constexpr int list_floats() { return DMAX == 0 ? 15360 : 4096; }

// The end of a round of `held` points, P to a team of `size` waves: the lanes' best meet in the waves, the waves' in LDS.
template <int DMAX, bool DIST, int P>
__device__ __forceinline__ void list_merge(
    const float* __restrict__ C, const int* ids, int64_t g, int len,
    int32_t* __restrict__ assign, float* __restrict__ min_dist, const float* xs, int d, int row_len, int K, int none, int size, int held,
    float (&best)[P], int (&at)[P], float (*cand_d)[8], int (*cand_k)[8]) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));                            // (or addresses made of it are kept through the round, in spilled registers)
    const int lane = tid & 63, wave = tid >> 6;
    // half of the lanes keep half of the points, then half of those, then the lanes of a point meet: ten exchanges for eight points where a
    // butterfly for each takes 48
    auto meet = [&](float d0, int k0, float d1, int k1, int o, int to) {     // (0: kept, 1: handed over)
        const float od = __shfl_xor(d1, o);
        const int ok = __shfl_xor(k1, o);
        const bool other = od < d0 || (od == d0 && ok < k0);
        best[to] = other ? od : d0;
        at[to] = other ? ok : k0;
    };
#pragma unroll
    for (int n = P / 2, o = 32; n > 0; n >>= 1, o >>= 1) {
        const bool upper = (lane & o) != 0;
#pragma unroll
        for (int p = 0; p < n; ++p)
            meet(upper ? best[n + p] : best[p], upper ? at[n + p] : at[p], upper ? best[p] : best[n + p], upper ? at[p] : at[n + p], o, p);
    }
#pragma unroll
    for (int o = 32 / P; o > 0; o >>= 1) meet(best[0], at[0], best[0], at[0], o, 0);
    if (lane % (64 / P) == 0) { cand_d[wave][lane * P / 64] = best[0]; cand_k[wave][lane * P / 64] = at[0]; }
    __syncthreads();
    if (tid < held && g + tid < len) {
        const int p = tid % P, w0 = tid / P * size;
        float bd = cand_d[w0][p];
        int bk = cand_k[w0][p];
        for (int w = w0 + 1; w < w0 + size; ++w) {
            const float od = cand_d[w][p];
            const int ok = cand_k[w][p];
            if (od < bd || (od == bd && ok < bk)) { bd = od; bk = ok; }
        }
        bk = bk < K ? bk : none;
        assign[ids[tid]] = bk;
        cand_k[w0][p] = bk;
    }
    __syncthreads();
    if constexpr (DIST) {
        const int here = (int)min((int64_t)held, len - g);
        auto measure = [&](auto group) {
            constexpr int LANES = decltype(group)::value, groups = 512 / LANES;
            for (int q0 = tid / LANES; q0 < here; q0 += 2 * groups) {        // (past the end: the last point again)
                const int q[2] = {q0, min(q0 + groups, here - 1)}, l = tid & (LANES - 1);
                const float* c[2];
                float D[2] = {0.f, 0.f};                     // (zeros past the end of both rows)
#pragma unroll
                for (int u = 0; u < 2; ++u) c[u] = C + (size_t)cand_k[q[u] / P * size][q[u] % P] * row_len;
                for (int j = l * 4; j < row_len; j += 4 * LANES) {
                    floatx4 w[2];
#pragma unroll
                    for (int u = 0; u < 2; ++u) w[u] = row_piece32(c[u], j, row_len);
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const floatx4 v = *(const floatx4*)(xs + q[u] * d + j);
#pragma unroll
                        for (int e = 0; e < 4; ++e) { const float t = v[e] - w[u][e]; D[u] = fmaf(t, t, D[u]); }
                    }
                }
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    D[u] = sum_of_lanes<LANES>(D[u]);
                    if (l == 0) min_dist[ids[q[u]]] = D[u];
                }
            }
        };
        if (DMAX == 32 && row_len <= 16) measure(std::integral_constant<int, 4>());
        else if (DMAX == 32) measure(std::integral_constant<int, 8>());
        else measure(std::integral_constant<int, 16>());
        __syncthreads();
    }
}

template <int DMAX, bool DIST, int P>
__device__ __forceinline__ void list_points(
    const float* __restrict__ X, const float* __restrict__ C, const int32_t* __restrict__ list, int len,
    int32_t* __restrict__ assign, float* __restrict__ min_dist, int d, int row_len, int K, int none, int teams, int G, float* xs, int* ids, float (*cand_d)[8], int (*cand_k)[8]) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int size = 8 / teams, team = wave / size, part = wave - team * size;   // waves of a team share the centroids
    const int held = teams * P;
    const float* x = xs + team * P * d;
    for (int64_t g = (int64_t)blockIdx.y * held; g < len; g += (int64_t)G * held) {
        // one wave per row (past the end of the list: the last point again)
        for (int r = wave; r < held; r += 8) {
            const int own = list[min(g + r, (int64_t)len - 1)];
            if (lane == 0) ids[r] = own;
            for (int j = lane * 4; j < d; j += 256) *(floatx4*)(xs + r * d + j) = row_piece32(X + (size_t)own * row_len, j, row_len);
        }
        float best[P];
        int at[P];
#pragma unroll
        for (int p = 0; p < P; ++p) { best[p] = INFINITY; at[p] = 0x7FFFFFFF; }
        __syncthreads();
        for (int k0 = part * 64; k0 < K; k0 += size * 64) {
            const int k = k0 + lane;
            const float* row = C + (size_t)min(k, K - 1) * row_len;
            float D[P];
#pragma unroll
            for (int p = 0; p < P; ++p) D[p] = 0.f;
            floatx4 c[8], next[8];                           // 32 features; d is a multiple of 8
            auto load = [&](floatx4 (&to)[8], int j) {
#pragma unroll
                for (int q = 0; q < 8; ++q) to[q] = raw_piece32(row, min(j + 4 * q, d - 4), row_len);
                if (j + 32 > row_len) {
#pragma unroll
                    for (int q = 0; q < 8; ++q) to[q] = settle32(to[q], min(j + 4 * q, d - 4), row_len);
                }
            };
            load(c, 0);
            for (int j0 = 0; j0 < d; j0 += 32) {
                if (j0 + 32 < d) load(next, j0 + 32);
#pragma unroll
                for (int q = 0; q < 8; q += 2) {
                    if (j0 + 4 * q < d) {
#pragma unroll
                        for (int p = 0; p < P; ++p) {
                            const floatx4 xa = *(const floatx4*)(x + p * d + j0 + 4 * q), xb = *(const floatx4*)(x + p * d + j0 + 4 * q + 4);
#pragma unroll
                            for (int e = 0; e < 4; ++e) { const float t = xa[e] - c[q][e]; D[p] = fmaf(t, t, D[p]); }
#pragma unroll
                            for (int e = 0; e < 4; ++e) { const float t = xb[e] - c[q + 1][e]; D[p] = fmaf(t, t, D[p]); }
                        }
                    }
                }
#pragma unroll
                for (int q = 0; q < 8; ++q) c[q] = next[q];
            }
            if (k < K) {
#pragma unroll
                for (int p = 0; p < P; ++p)
                    if (D[p] < best[p]) { best[p] = D[p]; at[p] = k; }
            }
        }
        list_merge<DMAX, DIST, P>(C, ids, g, len, assign, min_dist, xs, d, row_len, K, none, size, held, best, at, cand_d, cand_k);
    }
}

// Short lists of wide rows against many centroids: two points a team, lane = centroid row as in list_points, but the rows arrive 16
// features at a time in whole pieces of 64 bytes, two steps ahead (four or six: slower), and pass through LDS.  Read by their own lanes a
// step touches every line eight times, which a few workgroups alone feel: 11 points of d = 415 against 767 rows took 186 us,
// here 50.  Up to 256 centroids a wave has one block of rows, and the shorter chain of list_points is as fast or faster (fk_assign,
// us, this / that: 16000 points, d = 512, K = 230 60.6 / 55.2, d = 256, K = 100 36.2 / 34.3, d = 128, K = 200 27.7 / 29.2).
template <int DMAX, bool DIST>
__device__ __forceinline__ void list_few(
    const float* __restrict__ X, const float* __restrict__ C, const int32_t* __restrict__ list, int len,
    int32_t* __restrict__ assign, float* __restrict__ min_dist, int d, int row_len, int K, int none, int teams, int G, float* xs, float* tiles,
    int* ids, float (*cand_d)[8], int (*cand_k)[8]) {
    constexpr int P = 2, kRow = 20;                          // (four floats of padding: 16 lanes' reads hit all banks)
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int size = 8 / teams, team = wave / size, part = wave - team * size;
    const int held = teams * P, steps = (d + 15) / 16;
    const int blocks = K > part * 64 ? (K - part * 64 + size * 64 - 1) / (size * 64) : 0, all = blocks * steps;
    const float* x = xs + team * P * d;
    float* tile = tiles + wave * 64 * kRow;
    const int r0 = lane >> 2, j0 = (lane & 3) * 4;           // this lane's pieces: rows r0 + 16 q, features j0 .. j0 + 3
    for (int64_t g = (int64_t)blockIdx.y * held; g < len; g += (int64_t)G * held) {
        for (int r = wave; r < held; r += 8) {
            const int own = list[min(g + r, (int64_t)len - 1)];
            if (lane == 0) ids[r] = own;
            for (int j = lane * 4; j < d; j += 256) *(floatx4*)(xs + r * d + j) = row_piece32(X + (size_t)own * row_len, j, row_len);
        }
        float best[P], D[P];
        int at[P];
#pragma unroll
        for (int p = 0; p < P; ++p) { best[p] = INFINITY; at[p] = 0x7FFFFFFF; D[p] = 0.f; }
        __syncthreads();
        floatx4 ahead[2][4];
        uint32_t from[4];                                    // where this lane's rows of the block to load start (K len < 2^25)
        int load_block = 0, load_j = j0;
        auto load = [&](floatx4 (&to)[4]) {
            if (load_j == j0) {
#pragma unroll
                for (int q = 0; q < 4; ++q) from[q] = (uint32_t)min((part + load_block * size) * 64 + r0 + 16 * q, K - 1) * (uint32_t)row_len;
            }
            const int at_j = min(load_j, row_len - 4);       // (beyond the row: zeros, or nobody's)
#pragma unroll
            for (int q = 0; q < 4; ++q) to[q] = *(const floatx4_any*)(C + (from[q] + (uint32_t)at_j));
            if ((row_len & 7) && load_j + 4 > row_len) {
#pragma unroll
                for (int q = 0; q < 4; ++q) to[q] = settle32(to[q], load_j, row_len);
            }
            load_j += 16;
            if (load_j >= steps * 16) { load_j = j0; ++load_block; }
        };
        auto use = [&](floatx4 (&now)[4], int step, int block, int t) {
#pragma unroll
            for (int q = 0; q < 4; ++q) *(floatx4*)(tile + (r0 + 16 * q) * kRow + j0) = now[q];
            __builtin_amdgcn_wave_barrier();                 // LDS runs a wave's operations in order
            if (step + 2 < all) load(now);
#pragma unroll
            for (int e = 0; e < 16; e += 8) {                // (d is a multiple of 8)
                if (t * 16 + e < d) {
                    const floatx4 ca = *(const floatx4*)(tile + lane * kRow + e), cb = *(const floatx4*)(tile + lane * kRow + e + 4);
#pragma unroll
                    for (int p = 0; p < P; ++p) {
                        const floatx4 va = *(const floatx4*)(x + p * d + t * 16 + e), vb = *(const floatx4*)(x + p * d + t * 16 + e + 4);
#pragma unroll
                        for (int i = 0; i < 4; ++i) { const float u = va[i] - ca[i]; D[p] = fmaf(u, u, D[p]); }
#pragma unroll
                        for (int i = 0; i < 4; ++i) { const float u = vb[i] - cb[i]; D[p] = fmaf(u, u, D[p]); }
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();
            if (t + 1 == steps) {
                const int k = (part + block * size) * 64 + lane;
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    if (k < K && D[p] < best[p]) { best[p] = D[p]; at[p] = k; }
                    D[p] = 0.f;
                }
            }
        };
        if (all > 0) load(ahead[0]);
        if (all > 1) load(ahead[1]);
        for (int step = 0, block = 0, t = 0; step < all; step += 2) {
            use(ahead[0], step, block, t);
            if (++t == steps) { t = 0; ++block; }
            if (step + 1 < all) use(ahead[1], step + 1, block, t);
            if (++t == steps) { t = 0; ++block; }
        }
        list_merge<DMAX, DIST, P>(C, ids, g, len, assign, min_dist, xs, d, row_len, K, none, size, held, best, at, cand_d, cand_k);
    }
}

// Every lane's point `own`, whose centroid is k: the wave measures four a group of lanes at a time.
template <int LANES>
__device__ __forceinline__ void distances_of(const float* __restrict__ X, const float* __restrict__ C, float* __restrict__ min_dist, int own, int k, int len) {
    constexpr int U = 4, groups = 64 / LANES;
    const int lane = threadIdx.x & 63, l = lane & (LANES - 1);
    for (int p0 = lane / LANES; p0 < 64; p0 += U * groups) {
        int i[U];
        const float *x[U], *c[U];
        float s[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            i[u] = __shfl(own, p0 + u * groups);
            x[u] = X + (size_t)i[u] * len;
            c[u] = C + (size_t)__shfl(k, p0 + u * groups) * len;
        }
        row_distances<LANES, U>(x, c, len, l, s);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (l == 0) min_dist[i[u]] = s[u];
    }
}

template <int DMAX, bool DIST>
__device__ __forceinline__ void list_by_thread(
    const float* __restrict__ X, const float* __restrict__ C, const int32_t* __restrict__ list, int len,
    int32_t* __restrict__ assign, float* __restrict__ min_dist, int d, int row_len, int K, int none, int G, float* sc) {
    constexpr int TK = 32;
    for (int64_t g = (int64_t)blockIdx.y * 512; g < len; g += (int64_t)G * 512) {
        const int64_t at = g + threadIdx.x;
        const int own = list[min(at, (int64_t)len - 1)];
        float x[DMAX];
        load_row32<DMAX>(x, X + (size_t)own * row_len, row_len, true);
        float m = INFINITY;
        int a = none;
        for (int k0 = 0; k0 < K; k0 += TK) {
            __syncthreads();
            for (int o = threadIdx.x; o < TK * DMAX; o += 512) {
                const int r = o / DMAX, j = o % DMAX;
                sc[o] = (k0 + r < K && j < row_len) ? C[(size_t)(k0 + r) * row_len + j] : 0.f;
            }
            __syncthreads();
            const int nk = min(TK, K - k0);
            // (two chains at a time: a single one took 791 or 937 us, 200000 points, d = 64, K = 1000, every centroid twice, as the compiler
            // happened to choose registers; 714 so.  Past K the second one's row is zeros, and not looked at.)
            for (int r = 0; r < nk; r += 2) {
                float D[2] = {0.f, 0.f};
#pragma unroll
                for (int j = 0; j < DMAX; j += 4) {
                    const floatx4 c = *(const floatx4*)(sc + r * DMAX + j), c1 = *(const floatx4*)(sc + (r + 1) * DMAX + j);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float t = x[j + e] - c[e], t1 = x[j + e] - c1[e];
                        D[0] = fmaf(t, t, D[0]);
                        D[1] = fmaf(t1, t1, D[1]);
                    }
                }
                if (D[0] < m) { m = D[0]; a = k0 + r; }
                if (D[1] < m && r + 1 < nk) { m = D[1]; a = k0 + r + 1; }
            }
        }
        if (at < len) assign[own] = a;
        if constexpr (DIST) {
            // (past the end of the list: the last point again)
            if (DMAX == 32 && row_len <= 16) distances_of<4>(X, C, min_dist, own, a, row_len);
            else if (DMAX == 32) distances_of<8>(X, C, min_dist, own, a, row_len);
            else distances_of<16>(X, C, min_dist, own, a, row_len);
        }
    }
}

// Points that are open between two centroids, packed in assign: a wave takes as many as its part of LDS holds the
// differences to both of, in whole rows, and then has a lane add up the squares of each in the direct kernels' order.
// (From the last workgroup on: the first ones have the points that are measured in full.)
template <bool DIST>
__device__ __forceinline__ void list_pairs(
    const float* __restrict__ X, const float* __restrict__ C, const int32_t* __restrict__ list_end, int pairs,
    int32_t* __restrict__ assign, float* __restrict__ min_dist, int d, int row_len, int none, int G, float* diff, int floats) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, row = d + 4;     // (four floats: the lanes' reads spread over the banks)
    const int held = min((floats - 16) / (2 * row), 16);
    int* chosen = (int*)diff + floats - 16;
    const int waves = G * 8, each = min(held, (pairs + waves - 1) / waves);
    for (int64_t p0 = (int64_t)((G - 1 - blockIdx.y) * 8 + wave) * each; p0 < pairs; p0 += waves * each) {
        const int n = (int)min((int64_t)each, pairs - p0);
        const int own = list_end[-(p0 + min(lane, n - 1))];
        const uint32_t both = (uint32_t)(DIST ? __float_as_int(min_dist[own]) : assign[own]);
        const int k1 = (int)(both & 0xFFFFu), k2 = (int)(both >> 16);
        for (int p = 0; p < n; ++p) {
            const float* x = X + (size_t)__shfl(own, p) * row_len;
            const float *c1 = C + (size_t)__shfl(k1, p) * row_len, *c2 = C + (size_t)__shfl(k2, p) * row_len;
            for (int j = lane * 4; j < d; j += 256) {
                const floatx4 v = row_piece32(x, j, row_len), u1 = row_piece32(c1, j, row_len), u2 = row_piece32(c2, j, row_len);
                *(floatx4*)(diff + 2 * p * row + j) = v - u1;
                *(floatx4*)(diff + (2 * p + 1) * row + j) = v - u2;
            }
        }
        __builtin_amdgcn_wave_barrier();                     // LDS runs a wave's operations in order
        float D = 0.f;
        if (lane < 2 * n)
            for (int j = 0; j < d; j += 8) {
                const floatx4 a = *(const floatx4*)(diff + lane * row + j), c = *(const floatx4*)(diff + lane * row + j + 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) D = fmaf(a[e], a[e], D);
#pragma unroll
                for (int e = 0; e < 4; ++e) D = fmaf(c[e], c[e], D);
            }
        __builtin_amdgcn_wave_barrier();
        const float D1 = __shfl(D, 2 * lane), D2 = __shfl(D, 2 * lane + 1);
        if (lane < n) {
            // the lower centroid first, strict '<', from infinity: as the direct kernels go through them
            const int lo = min(k1, k2), hi = max(k1, k2);
            const float Dlo = k1 < k2 ? D1 : D2, Dhi = k1 < k2 ? D2 : D1;
            float best = INFINITY;
            int at = none;
            if (Dlo < best) { best = Dlo; at = lo; }
            if (Dhi < best) { best = Dhi; at = hi; }
            assign[own] = at;
            if (DIST) chosen[lane] = at;
        }
        if constexpr (DIST) {
            __builtin_amdgcn_wave_barrier();
            for (int p = lane >> 4; p < n; p += 4) {
                const int i = list_end[-(p0 + p)];
                const float* const x[1] = {X + (size_t)i * row_len};
                const float* const c[1] = {C + (size_t)chosen[p] * row_len};
                float s[1];
                row_distances<16, 1>(x, c, row_len, lane & 15, s);
                if ((lane & 15) == 0) min_dist[i] = s[0];
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
}

// `none`: the answer where no distance is finite, that of the direct kernel for the shape.
// DMAX: 32 or 64 for rows up to that, 0 for wider ones.  PAIRS: where the filter keeps three scores, DIST: where distances are wanted, and the
// code for either only there: with all of it in one kernel, and addresses of list_merge kept through its rounds, the long lists' registers did not
// suffice (four of each centroid, 2^20 points, d = 128, K = 64 943 us before pairs and distances had joined, 990 with them, 978 with the
// code apart, 871 with nothing spilled and the shorter merge; distances, once a pass of its own, 1050, 1211, 1169, 1007).
// The first G workgroups of an instance take the lists, the rest, where distances are wanted, measure the points that the
// filter has decided, in the time that the few open ones take.  A point that one of the lists has meanwhile given a centroid may be among
// them: both then write the same bits, and what the list still has to read of it (the two centroids, where its distance goes) it
// has read before it writes the centroid.
// The instances lie along x, so that the lists of all of them start before any measuring: one instance after the other the last
// one's list started last (fk_assign, distances, 32 instances of 19499 points, d = 39, K = 282 151 -> 132 us).
template <int DMAX, bool PAIRS, bool DIST>
__global__ __launch_bounds__(512, 4) void assign_f32_list_kernel(
    const float* __restrict__ X, const float* __restrict__ C, const int32_t* __restrict__ list,
    const int32_t* __restrict__ list_len, const int32_t* __restrict__ pair_len, int32_t* assign, float* min_dist, int64_t N, int d,
    int row_len, int K, int none, int G) {
    __shared__ __align__(16) float xs[list_floats<DMAX>()];
    __shared__ float cand_d[8][8];
    __shared__ int cand_k[8][8], ids[64];                    // (most points held: eight teams' eight)
    const int b = blockIdx.x;
    X += (size_t)b * N * row_len;
    C += (size_t)b * K * row_len;
    assign += (size_t)b * N;
    if (DIST) min_dist += (size_t)b * N;
    if (DIST && (int)blockIdx.y >= G) {
        const int64_t part = blockIdx.y - G, parts = gridDim.y - G;
        if (DMAX == 32 && row_len <= 16) measure_points<4, 4>(X, C, assign, min_dist, N, row_len, part, parts);
        else if (DMAX == 32) measure_points<8, 4>(X, C, assign, min_dist, N, row_len, part, parts);
        else if (DMAX == 64 || row_len <= 128) measure_points<16, 4>(X, C, assign, min_dist, N, row_len, part, parts);
        else measure_points<16, 2>(X, C, assign, min_dist, N, row_len, part, parts);
        return;
    }
    const int len = list_len[b];
    list += (size_t)b * N;
    const int most = K <= 64 ? 8 : K <= 128 ? 4 : K <= 256 ? 2 : 1;
    // waves with points of their own: where the centroids are too few to share, and where the list is long enough
    int thin = most, teams = 8;                              // both end at 1 or more (d <= 512)
    while (teams > most && len < teams * 8 * G) teams >>= 1;
    while (thin * 8 * d > 4096) thin >>= 1;                  // (short lists: as wide a spread)
    while (teams * 8 * d > list_floats<DMAX>()) teams >>= 1;
    if constexpr (PAIRS) {
        if (const int pairs = pair_len[b]; pairs > 0) {
            constexpr int kOwn = list_floats<DMAX>() / 8;
            list_pairs<DIST>(X, C, list + N - 1, pairs, assign, min_dist, d, row_len, none, G, xs + (threadIdx.x >> 6) * kOwn, kOwn);
            __syncthreads();
        }
    }
    if (len <= 2 * thin * G) {
        if constexpr (DMAX == 0) {
            if (K > 256) {
                list_few<DMAX, DIST>(X, C, list, len, assign, min_dist, d, row_len, K, none, thin, G, xs, xs + 4096, ids, cand_d, cand_k);
                return;
            }
        }
        list_points<DMAX, DIST, 2>(X, C, list, len, assign, min_dist, d, row_len, K, none, thin, G, xs, ids, cand_d, cand_k);
        return;
    }
    if constexpr (DMAX != 0) {
        if (len >= 256 * G && (K <= 128 || d > 16)) {
            list_by_thread<DMAX, DIST>(X, C, list, len, assign, min_dist, d, row_len, K, none, G, xs);
            return;
        }
    }
    list_points<DMAX, DIST, 8>(X, C, list, len, assign, min_dist, d, row_len, K, none, teams, G, xs, ids, cand_d, cand_k);
}

// ------------------------------------------------------------------------------------
static std::atomic<int> g_filter_option{-1};   // -1: by shape, 0: never, 1: always

void set_f32_filter_option(int v) { g_filter_option.store(v, std::memory_order_relaxed); }
int f32_filter_option() { return g_filter_option.load(std::memory_order_relaxed); }

// Where the filter wins, measured against the direct kernels over d = 16 .. 512, K = 8 .. 256 and
// 10^3 .. 2^20 points: its three launches take 18 us at least (20 with distances) and read X at the same rate, so the
// sweep has to be worth it.  Rows of up to 128: from 2^28 terms (32768 points, d = 128, K = 64: 19.1
// against 27.8 us; 131072, d = 64, K = 32: 21.7 against 27.7; below, 16384, d = K = 64: 19.2 against 13.5), or, with fewer
// points, where one wave's walk through the centroids alone is long enough (1000 points, d = 128, K = 64: 18.0
// against 22.2 us; d = 32, K = 128: 18.1 against 13.8).  (In a fit's later iterations it has two launches and would win
// sooner, which the rule does not tell apart: ten iterations there 164 against 213, 8192 points, d = 64, K = 100 268 against 324.)  Wider rows, which the direct kernel reads
// again for every 16 centroids: from the second such group (65536 points, d = 256, K = 512: 89
// against 1340 us), or with few points.
bool f32_filter_enabled(const Geometry& g) {
    const int opt = g.f32_filter;              // as it stood when the call began
    if (g.t != FK_F32 || opt == 0) return false;
    // two threads per point, and a launch dimension holds fewer than 2^32
    if (cdiv(g.N, 256) * 512 > (int64_t)UINT32_MAX) return false;
    if (opt > 0) return true;
    // On a line K clusters lie range / K apart: from about 64 the bound, some 2^-15 of the squared range, leaves
    // most points open (470330 points, d = 1, K = 918: 1011 us, the direct kernel 605; in a plane it pays:
    // 116170 points, d = 3, K = 581: 38 against 121).
    if (g.d_user == 1) return false;
    const int64_t points = (int64_t)g.B * g.N;
    if (g.d > 128) return g.K > 16 || points <= ((int64_t)1 << 16);
    return g.K >= 24 && (points * g.K * g.d >= ((int64_t)1 << 28) || g.K * std::max(g.d, 32) >= 8192);
}

template <int DCH>
static fk_status launch_filter_few(const Geometry& g, const Workspace& w, const float* X, int32_t* assign, float* min_dist, hipStream_t s) {
    hipLaunchKernelGGL(assign_f32_filter_few_kernel<DCH>, dim3((unsigned)cdiv(g.N, 32), g.B), dim3(kFewWaves * 64), 0, s, X,
                       (const uintx4*)w.c_frag, w.c_bias, w.f32_shift, assign, w.sorted_idx, w.f32_list_len, w.f32_pair_len, (int32_t*)min_dist,
                       g.N, g.d, g.len, g.K, g.ktiles);
    FK_HIP(hipGetLastError());
    return FK_OK;
}

template <int DCH, int WAVES>
static fk_status launch_filter_t(const Geometry& g, const Workspace& w, const float* X, int32_t* assign, float* min_dist, hipStream_t s) {
    dim3 grid((unsigned)cdiv(g.N, WAVES * 32), g.B), block(WAVES * 64);
    hipLaunchKernelGGL((assign_f32_filter_kernel<DCH, WAVES>), grid, block, 0, s, X, (const uintx4*)w.c_frag,
                       w.c_bias, w.f32_shift, assign, w.sorted_idx, w.f32_list_len, w.f32_pair_len, (int32_t*)min_dist, g.N, g.d, g.len, g.K, g.ktiles);
    FK_HIP(hipGetLastError());
    return FK_OK;
}

fk_status launch_f32_filter(const Geometry& g, const Workspace& w, const float* X, const float* C, int32_t* assign,
                            float* min_dist, F32Split split, hipStream_t s) {
    // (groups of eight features a thread, 32 rows of them to a workgroup)
    const int per = (int)cdiv(64 * g.dchunks, kLayoutThreads);
#define FK_LAYOUT(RAGGED) (per == 1 ? f32_split_layout_kernel<1, RAGGED> : per == 2 ? f32_split_layout_kernel<2, RAGGED> \
                           : per == 3 ? f32_split_layout_kernel<3, RAGGED> : f32_split_layout_kernel<4, RAGGED>)
    auto layout = g.len == g.d ? FK_LAYOUT(false) : FK_LAYOUT(true);
#undef FK_LAYOUT
    if (split != F32Split::kWritten) {
        hipLaunchKernelGGL(layout, dim3(g.ktiles, g.B), dim3(kLayoutThreads), 0, s, split == F32Split::kAmongPoints ? X : nullptr, (uint32_t)g.N, C, (uintx4*)w.c_frag, w.c_bias,
                           w.f32_shift, w.f32_list_len, w.f32_pair_len, g.d, g.len, g.K, g.ktiles, g.dchunks);
        FK_HIP(hipGetLastError());
    }
    // Workgroups of four waves fill the chip best; with very many points eight waves share each
    // copy of the centroids (2^20 points, 64 features, K = 256: 138 against 142 us; 128 features, K =
    // 64: 172 against 182 us) as long as two such workgroups fit a compute unit.
    // Few points (see assign_f32_filter_few_kernel), fk_assign, us, sweep / few: up to a tile of 32 points per compute unit always (1000, d = 64,
    // K = 200 22.4 / 20.0; five instances of 1516, d = 256, K = 12 in a fit 28.9 / 25.9), up to two where there are tiles of centroids to share
    // (16000, d = 256, K = 30 31.6 / 34.0; d = 96, K = 100 23.4 / 22.8; d = 256, K = 1000 93 / 77; d = 32, K = 8000 133 / 82); with 24000 points it
    // depends (d = 96, K = 1000 48 / 42, d = 256 92 / 94), with 32000 the sweep is faster (d = 128, K = 500 40.6 / 45.2).
    const int64_t tiles = cdiv(g.N, 32) * g.B;
    const bool few = tiles <= device_cu_count() || (tiles <= 2 * device_cu_count() && g.ktiles >= 4);
    const bool many = (int64_t)g.B * g.N >= ((int64_t)1 << 19);
#define FK_FILTER(DCH) \
    case DCH: \
        if (few) FK_TRY((launch_filter_few<DCH>(g, w, X, assign, min_dist, s))); \
        else if (DCH <= 8 && many) FK_TRY((launch_filter_t<DCH, DCH <= 8 ? 8 : 4>(g, w, X, assign, min_dist, s))); \
        else FK_TRY((launch_filter_t<DCH, 4>(g, w, X, assign, min_dist, s))); \
        break
    switch (g.dchunks) {
        FK_FILTER(1); FK_FILTER(2); FK_FILTER(3); FK_FILTER(4); FK_FILTER(5); FK_FILTER(6); FK_FILTER(7); FK_FILTER(8);
        FK_FILTER(10); FK_FILTER(12); FK_FILTER(14); FK_FILTER(16); FK_FILTER(20); FK_FILTER(24); FK_FILTER(28); FK_FILTER(32);
        default: set_error("fp32 assign: no kernel for %d feature chunks", g.dchunks); return FK_EUNSUPPORTED;
    }
#undef FK_FILTER
    const int64_t groups = cdiv(g.N, 2);
    const int64_t G = std::max<int64_t>(1, std::min<int64_t>(groups, cdiv((int64_t)device_cu_count() * 2, g.B)));
    const bool pairs = filter_keeps_three(g.dchunks);
#define FK_LIST(DIST) (g.d <= 32 ? assign_f32_list_kernel<32, false, DIST> : g.d <= 64 ? assign_f32_list_kernel<64, false, DIST> \
                       : pairs ? assign_f32_list_kernel<0, true, DIST> : assign_f32_list_kernel<0, false, DIST>)
    auto list_kernel = min_dist ? FK_LIST(true) : FK_LIST(false);
#undef FK_LIST
    int64_t distances = min_dist ? cdiv(f32_distance_blocks(g.N, distance_lanes(g.len)), g.d <= 128 ? 8 : 4) : 0;
    distances = std::min<int64_t>(distances, 16 * device_cu_count());      // (see measure_points)
    hipLaunchKernelGGL(list_kernel, dim3(g.B, (unsigned)(G + distances)), dim3(512), 0, s, X, C, w.sorted_idx,
                       w.f32_list_len, w.f32_pair_len, assign, min_dist, g.N, g.d, g.len, g.K, f32_direct_is_split(g) ? g.K - 1 : 0, (int)G);
    FK_HIP(hipGetLastError());
    return FK_OK;
}

}  // namespace fk
