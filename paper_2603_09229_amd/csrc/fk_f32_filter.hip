// fp32 assignment on the matrix cores, with the answer of the direct fp32 differences.
//
// Direct differences cost two vector instructions per (point, centroid, feature) and leave the
// matrix cores idle.  Here a first kernel only NARROWS the choice: it computes, for every pair,
//     s_k = x'.c'_k - |c'_k|^2 / 2          x' = x - m,  c' = c - m
// (the argmin of |x - c_k|^2 is the argmax of s_k; m, the mean of up to 32 of the centroids, keeps
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

// score bias that every real score loses to / that beats every real score; both are bf16 values
constexpr uint16_t kNever = 0xFF62, kAlways = 0x7F62;      // -/+ 3.0e38

__host__ __device__ constexpr float filter_kappa(int width) {
    return 7.62939453125e-06f + (0.53f * (float)width + 24.f) * 1.1920929e-07f;
}

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
// Tile 0 also leaves the shift m and clears the instance's list length.
// A few microseconds of dependent loads: the rows of the mean are asked for eight at a time and
// the own rows before the mean is needed.
constexpr int kLayoutThreads = 512;

__global__ __launch_bounds__(kLayoutThreads) void f32_split_layout_kernel(
    const float* __restrict__ C, uintx4* __restrict__ frag, float* __restrict__ c2,
    float* __restrict__ shift, int32_t* __restrict__ list_len, int d, int len, int K, int ktiles, int dch) {
    __shared__ float m[512];
    __shared__ double part[32][65];
    __shared__ int fits[32], odd_row[32];
    const int b = blockIdx.y, kt = blockIdx.x, tid = threadIdx.x;
    const int width = dch * 16;
    C += (size_t)b * K * len;
    frag += ((size_t)b * ktiles + kt) * (2 * dch + 1) * 64;
    // this thread's groups of eight features: group g = tid + i * threads is lane g % 64 of chunk g / 64
    constexpr int kGroups = 64 * 32 / kLayoutThreads;
    float own[kGroups][8];
#pragma unroll
    for (int i = 0; i < kGroups; ++i) {
        const int g = tid + i * kLayoutThreads;
        const int l = g & 63, k = kt * 32 + (l & 31), j0 = (g >> 6) * 16 + (l >> 5) * 8;
#pragma unroll
        for (int e = 0; e < 8; ++e) own[i][e] = 0.f;
        if (g < 64 * dch && k < K && j0 < d) {
            const floatx4 u = row_piece32(C + (size_t)k * len, j0, len), v = row_piece32(C + (size_t)k * len, j0 + 4, len);
#pragma unroll
            for (int e = 0; e < 4; ++e) { own[i][e] = u[e]; own[i][e + 4] = v[e]; }
        }
    }
    const int rows = min(K, 32);
    if (tid < width) {
        float s = 0.f;
        if (tid < len)
            for (int i0 = 0; i0 < rows; i0 += 8) {
                float v[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = C[(size_t)((int64_t)min(i0 + i, rows - 1) * K / rows) * len + tid];
#pragma unroll
                for (int i = 0; i < 8; ++i) s += i0 + i < rows && fabsf(v[i]) < INFINITY ? v[i] : 0.f;
            }
        s /= (float)rows;
        m[tid] = s;
        if (kt == 0) shift[(size_t)b * width + tid] = s;
    }
    if (tid < 32) odd_row[tid] = 0;
    if (kt == 0 && tid == 0) list_len[b] = 0;
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
    if (tid < 64) {
        const int r = tid & 31, h = tid >> 5, k = kt * 32 + r;
        double n2 = 0.0;
        for (int q = 0; q < 2 * dch; ++q) n2 += part[r][q];
        const bool never = k >= K || odd_row[r] != 0;
        const bool fine = !never && n2 < 1e38;               // false for NaN too
        uint16_t p[3] = {kNever, 0, 0};
        if (fine) {
            double left = (-0.5 + (double)filter_kappa(width)) * n2;
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                p[q] = float_to_lp((float)left, true);
                left -= (double)lp_to_float(p[q], true);
            }
        } else if (!never) {
            p[0] = kAlways;
        }
        uintx4 v = {0u, 0u, 0u, 0u};
        if (h == 0) {
            v[0] = (uint32_t)p[0] | ((uint32_t)p[1] << 16);
            v[1] = p[2];
            fits[r] = fine;
            c2[((size_t)b * ktiles + kt) * 32 + r] = fine ? (float)(n2 * 1.000001) : never ? 0.f : INFINITY;
        }
        frag[2 * dch * 64 + tid] = v;
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
    int32_t* __restrict__ list_len, int64_t N, int d, int len, int K, int ktiles) {
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

    float m1 = -INFINITY, m2 = -INFINITY;                    // best and second best, low 4 bits = 15 - slot
    int btile = 0;
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
        const float before = m1;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const float u = __uint_as_float((__float_as_uint(big[i] + small[i]) & 0xFFFFFFF0u) | (uint32_t)(15 - i));
            m2 = __builtin_amdgcn_fmed3f(m1, m2, u);
            m1 = __builtin_fmaxf(m1, u);
        }
        btile = m1 != before ? tile : btile;
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

    // the two lanes of a point meet
    const int i = 15 - (int)(__float_as_uint(m1) & 15u);
    int k = btile * 32 + 8 * (i >> 2) + 4 * h + (i & 3);
    const float o1 = __shfl_xor(m1, 32), o2 = __shfl_xor(m2, 32);
    const int ok = __shfl_xor(k, 32);
    x2 += __shfl_xor(x2, 32);
    m2 = __builtin_fmaxf(__builtin_fmaxf(m2, o2), __builtin_fminf(m1, o1));
    if (o1 > m1) { m1 = o1; k = ok; }
    k = min(k, K - 1);
    const float kappa = filter_kappa(DCH * 16);
    const float n2 = c2[k];
    const float room = 2.02f * kappa * (x2 + n2);
    // distance to the best one, from above (u_1 is s_1 + kappa |c'_1|^2 give or take room / 2)
    const float near = fmaxf(0.f, x2 - 2.f * m1) + 3.f * room;
    const float theta = (float)(d + 4) * 5.9604645e-08f * 1.1f * near;
    const bool certain = m1 - m2 > room + theta + 1e-30f;
    const bool mine = h == 0 && point < N;
    if (mine && certain) assign[point] = k;
    // A place on the list for the whole workgroup at once: additions to one address take 10 ns each, and
    // with many open points one per wave cost more than the sweep (2^20 points, all open: 330 us).
    // (The last stage has been read; LDS of its own would cost a workgroup per compute unit at DCH = 2.)
    int* opened = (int*)&even[0];
    int* list_at = opened + WAVES;
    const uint64_t open = __ballot(mine && !certain);
    if (lane == 0) opened[wave] = __popcll(open);
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        const int c = opened[w];
        before += w < wave ? c : 0;
        all += c;
    }
    if (all == 0) return;
    if (tid == 0) *list_at = atomicAdd(list_len + b, all);
    __syncthreads();
    if (mine && !certain) list[*list_at + before + __popcll(open & ((1ull << lane) - 1ull))] = (int32_t)point;
}

// The points on the list against all centroids by direct differences: ascending features, one
// fused multiply-add each, ascending centroids with strict '<' -- the same operations in the same
// order as assign_f32_kernel.
//   As a rule lane = centroid row, read 128 bytes at a time, a block of features ahead of its use;
// a wave holds P points.  The eight waves of a workgroup share out the centroids or, where those
// are too few, take points of their own (`teams` of 8 / teams waves each).  With P = 2 a short
// list is spread thin and over in the time that a few rows take to arrive (5 to 20 us); with P =
// 8 a long one is bound by the two vector instructions per term, as the direct kernels are.
//   Long lists of rows of up to 64 features, where that form spends its time on reading centroid
// rows: one point per thread with its features in registers, centroid tiles through LDS.  (Not rows of
// up to 16 against many centroids: it multiplies 32 features.  7 x 294694 points, d = 8, K = 14868: 60.1 ms
// against 34.4.)
//   What open points cost is then about the direct kernel's time for them on top of the filter's.
// Every centroid twice, so that all points are open, fk_assign against the direct kernels alone: 2^20 points,
// d = K = 64: 292 us, 222 (one addition to the list's length per wave: 610); d = 64, K = 256: 924, 814
// (in the first form: 1896); d = 128, K = 64: 950, 656 (4 teams: 1350); 300000 points, d = 96, K = 400:
// 1238, 1149; 65536, d = 256, K = 512: 696, 1323.

// Points held by a workgroup x row width, in floats.  Wide rows: enough that with few centroids as few
// waves as possible are without a share of them.
template <int DMAX>
constexpr int list_floats() { return DMAX == 0 ? 15360 : 4096; }

template <int P>
__device__ __forceinline__ void list_points(
    const float* __restrict__ X, const float* __restrict__ C, const int32_t* __restrict__ list, int len,
    int32_t* __restrict__ assign, int d, int row_len, int K, int none, int teams, float* xs, float (*cand_d)[8], int (*cand_k)[8]) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int size = 8 / teams, team = wave / size, part = wave - team * size;   // waves of a team share the centroids
    const int held = teams * P;
    const float* x = xs + team * P * d;
    for (int64_t g = (int64_t)blockIdx.x * held; g < len; g += (int64_t)gridDim.x * held) {
        // one wave per row (past the end of the list: the last point again)
        for (int r = wave; r < held; r += 8) {
            const int own = list[min(g + r, (int64_t)len - 1)];
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
#pragma unroll
        for (int p = 0; p < P; ++p) {
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                const float od = __shfl_xor(best[p], o);
                const int ok = __shfl_xor(at[p], o);
                if (od < best[p] || (od == best[p] && ok < at[p])) { best[p] = od; at[p] = ok; }
            }
            if (lane == 0) { cand_d[wave][p] = best[p]; cand_k[wave][p] = at[p]; }
        }
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
            assign[list[g + tid]] = bk < K ? bk : none;
        }
        __syncthreads();
    }
}

template <int DMAX>
__device__ __forceinline__ void list_by_thread(
    const float* __restrict__ X, const float* __restrict__ C, const int32_t* __restrict__ list, int len,
    int32_t* __restrict__ assign, int d, int row_len, int K, int none, float* sc) {
    constexpr int TK = 32;
    for (int64_t g = (int64_t)blockIdx.x * 512; g < len; g += (int64_t)gridDim.x * 512) {
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
            for (int r = 0; r < nk; ++r) {
                float D = 0.f;
#pragma unroll
                for (int j = 0; j < DMAX; j += 4) {
                    const floatx4 c = *(const floatx4*)(sc + r * DMAX + j);
#pragma unroll
                    for (int e = 0; e < 4; ++e) { const float t = x[j + e] - c[e]; D = fmaf(t, t, D); }
                }
                if (D < m) { m = D; a = k0 + r; }
            }
        }
        if (at < len) assign[own] = a;
    }
}

// `none`: the answer where no distance is finite, that of the direct kernel for the shape.
// DMAX: 32 or 64 for rows up to that, 0 for wider ones.
template <int DMAX>
__global__ __launch_bounds__(512, 4) void assign_f32_list_kernel(
    const float* __restrict__ X, const float* __restrict__ C, const int32_t* __restrict__ list,
    const int32_t* __restrict__ list_len, int32_t* __restrict__ assign, int64_t N, int d, int row_len,
    int K, int none) {
    __shared__ __align__(16) float xs[list_floats<DMAX>()];
    __shared__ float cand_d[8][8];
    __shared__ int cand_k[8][8];
    const int b = blockIdx.y;
    const int len = list_len[b];
    X += (size_t)b * N * row_len;
    C += (size_t)b * K * row_len;
    assign += (size_t)b * N;
    list += (size_t)b * N;
    const int most = K <= 64 ? 8 : K <= 128 ? 4 : K <= 256 ? 2 : 1;
    int thin = most, teams = most;                           // both end at 1 or more (d <= 512)
    while (thin * 8 * d > 4096) thin >>= 1;                  // (short lists: as wide a spread)
    while (teams * 8 * d > list_floats<DMAX>()) teams >>= 1;
    if (len <= 2 * thin * (int)gridDim.x)
        list_points<2>(X, C, list, len, assign, d, row_len, K, none, thin, xs, cand_d, cand_k);
    else if (DMAX == 0 || len < 256 * (int)gridDim.x || (K > 128 && d <= 16))
        list_points<8>(X, C, list, len, assign, d, row_len, K, none, teams, xs, cand_d, cand_k);
    else
        list_by_thread<DMAX == 0 ? 32 : DMAX>(X, C, list, len, assign, d, row_len, K, none, xs);
}

// min_dist[i] = |x_i - c_a(i)|^2 by direct differences: LANES (4, 8 or 16) lanes a point, enough for a whole
// row per load where it has up to 64 features.  Infinity where it is not finite, as in the direct
// kernels, whose minimum starts there.  (The lanes' sums meet in a butterfly: lanes without a piece add
// zero, so that their number changes no bit.)
template <int LANES>
__global__ __launch_bounds__(256) void f32_distance_kernel(
    const float* __restrict__ X, const float* __restrict__ C, const int32_t* __restrict__ assign,
    float* __restrict__ min_dist, int64_t N, int len, int K) {
    const int b = blockIdx.y, l = threadIdx.x & (LANES - 1);
    constexpr int kPoints = 256 / LANES;
    for (int64_t i = (int64_t)blockIdx.x * kPoints + threadIdx.x / LANES; i < N; i += (int64_t)gridDim.x * kPoints) {
        const float* x = X + ((size_t)b * N + i) * len;
        const float* c = C + ((size_t)b * K + assign[(size_t)b * N + i]) * len;
        float s = 0.f;
        for (int j = l * 4; j < len; j += 4 * LANES) {
            const floatx4 u = row_piece32(x, j, len), v = row_piece32(c, j, len);
#pragma unroll
            for (int e = 0; e < 4; ++e) { const float t = u[e] - v[e]; s = fmaf(t, t, s); }
        }
#pragma unroll
        for (int o = LANES / 2; o > 0; o >>= 1) s += __shfl_xor(s, o);   // (the lanes of a point leave together)
        if (l == 0) min_dist[(size_t)b * N + i] = s < INFINITY ? s : INFINITY;
    }
}

// ------------------------------------------------------------------------------------
static std::atomic<int> g_filter_option{-1};   // -1: by shape, 0: never, 1: always

void set_f32_filter_option(int v) { g_filter_option.store(v, std::memory_order_relaxed); }

// Where the filter wins, measured against the direct kernels over d = 16 .. 512, K = 8 .. 256 and
// 10^3 .. 2^20 points: its three launches take 14 us at least and read X at the same rate, so the
// sweep has to be worth it.  Rows of up to 128: from 2^28 terms (32768 points, d = 128, K = 64: 21.1
// against 27.2 us; 131072, d = 64, K = 32: 20.1 against 29.1), or, with fewer points, where one
// wave's walk through the centroids alone is long enough (1000 points, d = 128, K = 64: 19.4
// against 22.1 us; d = 32, K = 128: 15.4 against 13.9).  Wider rows, which the direct kernel reads
// again for every 16 centroids: from the second such group (65536 points, d = 256, K = 512: 89
// against 1340 us), or with few points.
bool f32_filter_enabled(const Geometry& g) {
    const int opt = g_filter_option.load(std::memory_order_relaxed);
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

template <int DCH, int WAVES>
static fk_status launch_filter_t(const Geometry& g, const Workspace& w, const float* X, int32_t* assign, hipStream_t s) {
    dim3 grid((unsigned)cdiv(g.N, WAVES * 32), g.B), block(WAVES * 64);
    hipLaunchKernelGGL((assign_f32_filter_kernel<DCH, WAVES>), grid, block, 0, s, X, (const uintx4*)w.c_frag,
                       w.c_bias, w.f32_shift, assign, w.sorted_idx, w.f32_list_len, g.N, g.d, g.len, g.K, g.ktiles);
    FK_HIP(hipGetLastError());
    return FK_OK;
}

fk_status launch_f32_filter(const Geometry& g, const Workspace& w, const float* X, const float* C, int32_t* assign,
                            float* min_dist, hipStream_t s) {
    hipLaunchKernelGGL(f32_split_layout_kernel, dim3(g.ktiles, g.B), dim3(kLayoutThreads), 0, s, C, (uintx4*)w.c_frag, w.c_bias,
                       w.f32_shift, w.f32_list_len, g.d, g.len, g.K, g.ktiles, g.dchunks);
    FK_HIP(hipGetLastError());
    // Workgroups of four waves fill the chip best; with very many points eight waves share each
    // copy of the centroids (2^20 points, 64 features, K = 256: 138 against 142 us; 128 features, K =
    // 64: 172 against 182 us) as long as two such workgroups fit a compute unit.
    const bool many = (int64_t)g.B * g.N >= ((int64_t)1 << 19);
#define FK_FILTER(DCH) \
    case DCH: \
        if (DCH <= 8 && many) FK_TRY((launch_filter_t<DCH, DCH <= 8 ? 8 : 4>(g, w, X, assign, s))); \
        else FK_TRY((launch_filter_t<DCH, 4>(g, w, X, assign, s))); \
        break
    switch (g.dchunks) {
        FK_FILTER(1); FK_FILTER(2); FK_FILTER(3); FK_FILTER(4); FK_FILTER(5); FK_FILTER(6); FK_FILTER(7); FK_FILTER(8);
        FK_FILTER(10); FK_FILTER(12); FK_FILTER(14); FK_FILTER(16); FK_FILTER(20); FK_FILTER(24); FK_FILTER(28); FK_FILTER(32);
        default: set_error("fp32 assign: no kernel for %d feature chunks", g.dchunks); return FK_EUNSUPPORTED;
    }
#undef FK_FILTER
    const int64_t groups = cdiv(g.N, 2);
    const int64_t G = std::max<int64_t>(1, std::min<int64_t>(groups, cdiv((int64_t)device_cu_count() * 2, g.B)));
    auto list_kernel = g.d <= 32 ? assign_f32_list_kernel<32> : g.d <= 64 ? assign_f32_list_kernel<64>
                                                                          : assign_f32_list_kernel<0>;
    hipLaunchKernelGGL(list_kernel, dim3((unsigned)G, g.B), dim3(512), 0, s, X, C, w.sorted_idx,
                       w.f32_list_len, assign, g.N, g.d, g.len, g.K, f32_direct_is_split(g) ? g.K - 1 : 0);
    FK_HIP(hipGetLastError());
    if (min_dist) {
        const int lanes = g.d <= 16 ? 4 : g.d <= 32 ? 8 : 16;
        auto kern = lanes == 4 ? f32_distance_kernel<4> : lanes == 8 ? f32_distance_kernel<8> : f32_distance_kernel<16>;
        hipLaunchKernelGGL(kern, dim3((unsigned)f32_distance_blocks(g.N, lanes), g.B), dim3(256), 0, s, X, C, assign,
                           min_dist, g.N, g.len, g.K);
        FK_HIP(hipGetLastError());
    }
    return FK_OK;
}

}  // namespace fk
