// Few clusters (K <= 32, 16-bit storage, d <= 128): the centroid update without any sort or
// gather, optionally fused into the assignment pass.
//
// With so few clusters the update of Section 4.2 spends its time re-reading X through the
// sorted index; the whole table of sums is only K x d floats.  Here every wave keeps that
// table in MFMA accumulators and adds a batch of 32 points to it with one more contraction:
//     S[k][j] += sum_p onehot[k][p] * x[p][j],   onehot[k][p] = (a_p == k)
// The products are exact (x times 1 or 0) and accumulate in fp32, so this is Eq. 3's sum in a
// fixed, reproducible order -- no atomics, as in the sort-inverse path.  X is streamed once,
// row-contiguous; when the assignment is computed in the same pass (ASSIGN), one Lloyd
// iteration reads X once instead of twice.  The contraction runs over points, so its
// X-operand is the transpose of the batch as it sits in LDS: it is read with the
// transposing LDS load (each lane receives four consecutive points of one feature column).
//
// Every workgroup leaves one partial table and one count per cluster; the ordinary
// merge/normalise kernel adds a cluster's partial rows (and counts) in workgroup order.
//
// What bounds it: reading X.  2^24 points, d = 64, K = 16 (2 GiB), us per iteration in a fit, merge included: 420 as it was
// (5.2 TB/s), 389 with copies that ask for no place in the caches, 372 with less of X in flight (stream_per_cu) and half the vector
// instructions, 318 where the assignment is not written: 64 MiB of stores among the reads cost 60 us, so only the
// iteration whose assignment the caller sees writes it (about 5% less with the hint on the stores too).  A contiguous
// share of X per workgroup instead of batches in turn: 403 for 393, 331 for 326 in fk_update.  Where X is small it is a chain of latencies:
// 300000 points, d = 64, K = 16 21.0 -> 16.1 us, 14324, d = 128, K = 14 13.1 -> 11.7.
#include <algorithm>

#include "fk_common.h"
#include "fk_device.h"

namespace fk {

// X is read once: copies of whole lines that ask for no place in the caches (the non-temporal hint).
constexpr int kOnce = 2;

// Workgroups per compute unit: no more than keep 32 KiB of X in flight there, 64 where rows of 64 features are assigned too and of wider rows.  More make memory
// slower, and the merge longer.  fk_update, us, one / two / three: 2^24 points, d = 64, K = 16 309 / 327 / 354; 8 million, d = 128, K = 30
// 306 / 319; 16 million, d = 32, K = 30 204 / 165 / 186.  An iteration: 2^20, d = 128, K = 32 52 / 57; 3 million, d = 48, K = 12 63 / 54 /
// 58 (one wave per SIMD is too few for the work on rows that are not swizzled); 16 million, d = 32 238 / 175 / 172; 200000, d = 32,
// K = 32 12.7 / 13.0 / 14.3.  (Rows of 40 features, which are not stored swizzled and of which one has 20 KiB in flight, always take two: fk_update,
// K = 20, one / two: 60 MB of them 22 / 20, 260 MB 56 / 51, 1200 MB 217 / 192; rows of 48 take as long either way.)
constexpr int stream_per_cu(int dch, bool assigns) { return dch == 8 || (dch == 4 && !assigns) ? 1 : 2; }

// Few workgroups make a wave's share long, 16384 of 2^24 points, and one chain of additions over all of it loses what is small
// beside its sum: some 1e-5 of a mean of ones and a few values of 2^-11 (test_long_chains in tests/test_gpu_few_clusters.py); 2.2e-7 of one of
// normally distributed numbers about zero, 1.4e-7 with three times as many workgroups, 1.2e-7 so: where a wave has more than this many batches,
// sums of so many are added up in a second set of registers.  fk_update, 2^24 points, d = 64, K = 16 308.4 us without and with it, d = 32, K = 30 171.8
// and 172.6; two iterations there 367 and 371.  (Rows of 128 features that are assigned too leave no registers: one workgroup a unit, as always.)
constexpr int kStreamRun = 32;

// BF: bf16 (else fp16).  DCH: feature chunks of 16 per point (2, 4 or 8).  ASSIGN: compute
// the assignment here (argmax of x.c_k - ||c_k||^2/2 over the single centroid tile, same
// packed-score rules as the assignment kernels) and, where `keep` says so, write it; otherwise read it.
//
// Grid (G, B).  Wave w of workgroup g handles the 32-point batches g*WAVES + w,
// + G*WAVES, ...: a fixed partition, so the partial tables are reproducible.
// partial: [B][K][G][d] floats, wg_counts: [B][K][G].
// RUNS: sums of kStreamRun batches at a time, and of those.
template <bool BF, int DCH, int WAVES, bool ASSIGN, bool RUNS>
__global__ __launch_bounds__(WAVES * 64, stream_per_cu(DCH, ASSIGN)) void stream_update_kernel(
    const uint16_t* __restrict__ X, const uintx4* __restrict__ c_frag,
    const float* __restrict__ c_bias, int32_t* assign, float* __restrict__ partial,
    int32_t* __restrict__ wg_counts, int64_t N, int d, int K, int keep) {
    constexpr int kThreads = WAVES * 64;
    constexpr int kRows = 32;                          // points per batch
    constexpr int CB = DCH / 2;                        // 32-feature column blocks of the table
    constexpr int kIdVec = ASSIGN ? 0 : 16;            // 256 bytes of cluster ids behind a batch
    constexpr int kBufVec = DCH * 64 + kIdVec;         // 16-byte vectors per batch buffer
    constexpr int loads = DCH + (ASSIGN ? 0 : 1);      // copy instructions per batch, always all issued
    constexpr uint32_t kOne = BF ? 0x3F80u : 0x3C00u;  // 1.0 in the storage type
    extern __shared__ uintx4 dyn_lds[];                // per wave: two batch buffers
    const int ppr = d >> 3;                            // 16-byte pieces per row
    const int swz = (ppr & (ppr - 1)) == 0 ? min(ppr, 8) - 1 : 0;   // XOR mask for the piece index

    const int b = blockIdx.y, G = gridDim.x, wg = blockIdx.x;
    X += (size_t)b * N * d;
    assign += (size_t)b * N;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, h = lane >> 5;
    uintx4* ring = dyn_lds + (size_t)wave * 2 * kBufVec;

    const int64_t nbatches = (N + kRows - 1) / kRows;
    const int64_t stride = (int64_t)G * WAVES;
    int64_t t = (int64_t)wg * WAVES + wave;

    // Slot j of a buffer holds piece (j % ppr) ^ (row & swz) of row j / ppr.  Every copy
    // instruction is issued with all lanes live (rows past the end of X or of the batch
    // re-read the last valid row): the waits below count instructions, and a stale slot
    // must hold finite values because it is multiplied by a zero of the one-hot operand.
    // A lane's places in a batch are the same for every batch but the one that X ends in.
    uint32_t from[DCH];
#pragma unroll
    for (int q = 0; q < DCH; ++q) {
        const int j = q * 64 + lane, row = j / ppr;
        from[q] = (uint32_t)min(row, kRows - 1) * (uint32_t)d * 2u + (uint32_t)(((j - row * ppr) ^ (row & swz)) << 4);
    }
    auto request = [&](int64_t batch, uintx4* buf) {
        const char* at = (const char*)X + (size_t)batch * (kRows * 2) * d;
        const int rows = (int)min((int64_t)kRows, N - batch * kRows);
        uint32_t o[DCH];
#pragma unroll
        for (int q = 0; q < DCH; ++q) o[q] = from[q];
        if (rows < kRows) {
#pragma unroll
            for (int q = 0; q < DCH; ++q) o[q] -= (uint32_t)max(0, min((q * 64 + lane) / ppr, kRows - 1) - (rows - 1)) * (uint32_t)d * 2u;
        }
#pragma unroll
        for (int q = 0; q < DCH; ++q)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(at + o[q]),
                                             (__attribute__((address_space(3))) void*)(buf + q * 64), 16, 0, kOnce);
        if (!ASSIGN)
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void*)(assign + batch * kRows + min(lane, rows - 1)),
                (__attribute__((address_space(3))) void*)(buf + DCH * 64), 4, 0, kOnce);
    };
    // the centroids (A operands) and their bias stay in registers
    uintx4 cf[ASSIGN ? DCH : 1];
    floatx16 bias16;
    if (ASSIGN) {
        c_frag += (size_t)b * DCH * 64;
        c_bias += (size_t)b * 32;
#pragma unroll
        for (int s = 0; s < DCH; ++s) cf[s] = c_frag[s * 64 + lane];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const floatx4 bv = *(const floatx4*)&c_bias[8 * q + 4 * h];
#pragma unroll
            for (int e = 0; e < 4; ++e) bias16[4 * q + e] = bv[e];
        }
    }
    if (t < nbatches) request(t, ring);
    if (t + stride < nbatches) request(t + stride, ring + kBufVec);
    if (ASSIGN) {
        // (waited for here, or the compiler waits for them, and with them for younger copies, in the loop)
#pragma unroll
        for (int s = 0; s < DCH; ++s) asm volatile("" : "+v"(cf[s]));
        asm volatile("" : "+v"(bias16));
    }

    // Where this lane reads: its B operands, features [16 s + 8 h, + 8) of point n (chunks past d meet zero
    // centroid features), and its share of the transposing reads.  Inside a group of 16 lanes, lane L
    // supplies the 8 bytes (row L/4, columns 4*(L%4)..+3) of a 4 x 16 block and receives
    // column L of it.  Group (lane/16): bit 0 = which 16 columns of the 32, bit 1 = h.
    const int L = lane & 15, nb = (lane >> 4) & 1;
    uint32_t x_at[ASSIGN ? DCH : 1], t_at[2][CB][2];
    if (ASSIGN)
#pragma unroll
        for (int s = 0; s < DCH; ++s) x_at[s] = (uint32_t)(n * ppr + (min(2 * s + h, ppr - 1) ^ (n & swz))) << 4;
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int row = 16 * s2 + 8 * h + 4 * u + (L >> 2);
                t_at[s2][cb][u] = ((uint32_t)(row * ppr + (min(4 * cb + 2 * nb + ((L & 3) >> 1), ppr - 1) ^ (row & swz))) << 4) + ((L & 1) << 3);
            }

    floatx16 accS[CB], whole[RUNS ? CB : 1];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) accS[cb] = whole[RUNS ? cb : 0] = floatx16{};
    int cnt = 0, run = 0;

    // A batch is read into registers as a whole, so that its buffer takes the batch after the next at once: two
    // batches are in flight while one is worked on (a third buffer, filled an iteration later, kept as many).  Copies and stores of a
    // wave complete in order; behind the copies of the batch that is waited for there are those of the next one and, from the
    // second batch on, the store of the one before.
    if (t + stride < nbatches) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(loads) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

    int cur = 0;
    while (t < nbatches) {
        uintx4* bufc = ring + cur * kBufVec;
        const uint32_t at = lds_addr(bufc);

        // LDS reads through opaque instructions: the wait for the copy that filled this buffer
        // was issued by hand, and the compiler must not add one for the younger copy in flight.
        // Every group of reads sits in ONE asm statement together with its wait, with all its
        // results as outputs: no result register can be touched between issue and arrival.
        uintx4 xf[ASSIGN ? DCH : 1];
        if (ASSIGN) {
            uint32_t xa[DCH];
#pragma unroll
            for (int s = 0; s < DCH; ++s) xa[s] = at + x_at[s];
            if constexpr (DCH == 2)
                asm volatile("ds_read_b128 %0, %2\n\tds_read_b128 %1, %3\n\ts_waitcnt lgkmcnt(0)"
                             : "=&v"(xf[0]), "=&v"(xf[1]) : "v"(xa[0]), "v"(xa[1]) : "memory");
            else if constexpr (DCH == 4)
                asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\t"
                             "ds_read_b128 %3, %7\n\ts_waitcnt lgkmcnt(0)"
                             : "=&v"(xf[0]), "=&v"(xf[1]), "=&v"(xf[2]), "=&v"(xf[3])
                             : "v"(xa[0]), "v"(xa[1]), "v"(xa[2]), "v"(xa[3]) : "memory");
            else {
                static_assert(DCH == 2 || DCH == 4 || DCH == 8, "feature chunks per point");
                asm volatile("ds_read_b128 %0, %8\n\tds_read_b128 %1, %9\n\tds_read_b128 %2, %10\n\t"
                             "ds_read_b128 %3, %11\n\tds_read_b128 %4, %12\n\tds_read_b128 %5, %13\n\t"
                             "ds_read_b128 %6, %14\n\tds_read_b128 %7, %15\n\ts_waitcnt lgkmcnt(0)"
                             : "=&v"(xf[0]), "=&v"(xf[1]), "=&v"(xf[2]), "=&v"(xf[3]), "=&v"(xf[4 % DCH]), "=&v"(xf[5 % DCH]),
                               "=&v"(xf[6 % DCH]), "=&v"(xf[7 % DCH])
                             : "v"(xa[0]), "v"(xa[1]), "v"(xa[2]), "v"(xa[3]), "v"(xa[4 % DCH]), "v"(xa[5 % DCH]),
                               "v"(xa[6 % DCH]), "v"(xa[7 % DCH]) : "memory");
            }
        }
        // transposed operand: one statement (reads + wait) per pair of column blocks
        uintx2 xt[2][CB][2];
        if constexpr (CB == 1) {
            asm volatile("ds_read_b64_tr_b16 %0, %4\n\tds_read_b64_tr_b16 %1, %5\n\t"
                         "ds_read_b64_tr_b16 %2, %6\n\tds_read_b64_tr_b16 %3, %7\n\ts_waitcnt lgkmcnt(0)"
                         : "=&v"(xt[0][0][0]), "=&v"(xt[0][0][1]), "=&v"(xt[1][0][0]), "=&v"(xt[1][0][1])
                         : "v"(at + t_at[0][0][0]), "v"(at + t_at[0][0][1]), "v"(at + t_at[1][0][0]), "v"(at + t_at[1][0][1])
                         : "memory");
        } else {
#pragma unroll
            for (int cb = 0; cb < CB; cb += 2) {
                uint32_t ta[2][2][2];
#pragma unroll
                for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
                    for (int c = 0; c < 2; ++c)
#pragma unroll
                        for (int u = 0; u < 2; ++u) ta[s2][c][u] = at + t_at[s2][(cb + c) % CB][u];
                asm volatile("ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %1, %9\n\t"
                             "ds_read_b64_tr_b16 %2, %10\n\tds_read_b64_tr_b16 %3, %11\n\t"
                             "ds_read_b64_tr_b16 %4, %12\n\tds_read_b64_tr_b16 %5, %13\n\t"
                             "ds_read_b64_tr_b16 %6, %14\n\tds_read_b64_tr_b16 %7, %15\n\ts_waitcnt lgkmcnt(0)"
                             : "=&v"(xt[0][cb][0]), "=&v"(xt[0][cb][1]), "=&v"(xt[0][(cb + 1) % CB][0]), "=&v"(xt[0][(cb + 1) % CB][1]),
                               "=&v"(xt[1][cb][0]), "=&v"(xt[1][cb][1]), "=&v"(xt[1][(cb + 1) % CB][0]), "=&v"(xt[1][(cb + 1) % CB][1])
                             : "v"(ta[0][0][0]), "v"(ta[0][0][1]), "v"(ta[0][1][0]), "v"(ta[0][1][1]),
                               "v"(ta[1][0][0]), "v"(ta[1][0][1]), "v"(ta[1][1][0]), "v"(ta[1][1][1])
                             : "memory");
            }
        }
        int k = 0;
        if (!ASSIGN)
            asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)"
                         : "=&v"(k) : "v"(at + DCH * 1024 + (uint32_t)(n << 2)) : "memory");

        const int64_t t1 = t + stride, t2 = t1 + stride;
        const bool issued = t2 < nbatches;
        if (issued) request(t2, bufc);

        const int rows = (int)min((int64_t)kRows, N - t * kRows);
        if (ASSIGN) {
            floatx16 acc = mfma32<BF>(cf[0], xf[0], bias16);
#pragma unroll
            for (int s = 1; s < DCH; ++s) acc = mfma32<BF>(cf[s], xf[s], acc);
            // score with its low 4 mantissa bits replaced by 15 - slot: one max carries both
            float m = -INFINITY;
#pragma unroll
            for (int i = 0; i < 16; i += 2) {
                const float k0 = __uint_as_float((__float_as_uint(acc[i]) & 0xFFFFFFF0u) | (uint32_t)(15 - i));
                const float k1 = __uint_as_float((__float_as_uint(acc[i + 1]) & 0xFFFFFFF0u) | (uint32_t)(14 - i));
                m = __builtin_fmaxf(__builtin_fmaxf(m, k0), k1);
            }
            const uint32_t bits = __float_as_uint(m);
            const int i = 15 - (int)(bits & 15u);
            k = 8 * (i >> 2) + 4 * h + (i & 3);
            // both lanes of a point see what the lower and the upper one have found
            const uintx2 ms = __builtin_amdgcn_permlane32_swap(bits & 0xFFFFFFF0u, bits & 0xFFFFFFF0u, false, false);
            const uintx2 ks = __builtin_amdgcn_permlane32_swap((uint32_t)k, (uint32_t)k, false, false);
            const float m0 = __uint_as_float(ms[0]), m1 = __uint_as_float(ms[1]);
            const bool upper = m1 > m0 || (m1 == m0 && ks[1] < ks[0]);
            k = min((int)(upper ? ks[1] : ks[0]), K - 1);
            if (keep && lane < rows) __builtin_nontemporal_store(k, &assign[t * kRows + lane]);
        } else {
            k = min(max(k, 0), K - 1);
        }

        // one-hot rows: bit p of E says that point p of the batch belongs to cluster n (this
        // lane's row of the table), built from the bit planes of the 32 cluster ids
        uint32_t E = 0xFFFFFFFFu >> (kRows - rows);
#pragma unroll
        for (int bit = 0; bit < 5; ++bit) {
            const uint32_t pl = (uint32_t)__ballot((k >> bit) & 1);
            E &= ((n >> bit) & 1) ? pl : ~pl;
        }
        cnt += __popc(E);
        E >>= 8 * h;
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
            // even points' bits stay where they are, odd ones' go 15 places up: points 2 q and 2 q + 1 are then bits
            // 2 q and 2 q + 16, which one product turns into a pair of ones (kOne is a multiple of 64)
            const uint32_t byte = E >> (16 * s2), spread = (byte & 0x55u) | ((byte & 0xAAu) << 15);
            uintx4 A;
#pragma unroll
            for (int q = 0; q < 4; ++q) A[q] = __umul24(spread & (0x10001u << (2 * q)), kOne >> (2 * q));
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                const uintx4 Bt = {xt[s2][cb][0][0], xt[s2][cb][0][1], xt[s2][cb][1][0], xt[s2][cb][1][1]};
                accS[cb] = mfma32<BF>(A, Bt, accS[cb]);
            }
        }
        if (RUNS && ++run == kStreamRun) {
            run = 0;
            asm volatile("");                          // (a branch, or the compiler selects in every batch)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) { whole[RUNS ? cb : 0] += accS[cb]; accS[cb] = floatx16{}; }
        }

        // the next batch must have landed before it is read (wave-private buffers: no barrier)
        if (issued && ASSIGN && keep) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(loads + 1) : "memory");
        else if (issued) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(loads) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        t = t1;
        cur ^= 1;
    }

    // The waves' tables meet in LDS (the ring is free now) and are added in wave order.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    constexpr int dpad = DCH * 16;
    float* comb = (float*)dyn_lds;                     // [WAVES][32][dpad]
    int* ccnt = (int*)(comb + WAVES * 32 * dpad);      // [WAVES][32]
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int i = 0; i < 16; ++i)
            comb[(wave * 32 + 8 * (i >> 2) + 4 * h + (i & 3)) * dpad + 32 * cb + n] = RUNS ? whole[RUNS ? cb : 0][i] + accS[cb][i] : accS[cb][i];
    if (h == 0) ccnt[wave * 32 + n] = cnt;
    __syncthreads();
    for (int o = tid; o < K * d; o += kThreads) {
        const int kk = o / d, j = o - kk * d;
        float s = comb[kk * dpad + j];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) s += comb[(w * 32 + kk) * dpad + j];
        partial[(((size_t)b * K + kk) * G + wg) * d + j] = s;
    }
    if (tid < K) {
        int c = 0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) c += ccnt[w * 32 + tid];
        wg_counts[((size_t)b * K + tid) * G + wg] = c;
    }
}

// ------------------------------------------------------------------------------------
static std::atomic<int> g_fused_option{-1};   // -1 / 1: use when the shape allows, 0: never

void set_fused_update_option(int v) { g_fused_option.store(v, std::memory_order_relaxed); }

bool fused_update_allowed() { return g_fused_option.load(std::memory_order_relaxed) != 0; }

template <bool BF, int DCH, bool ASSIGN>
static fk_status launch_stream_update_t(const Geometry& g, const Workspace& w, const void* X,
                                        int32_t* assign, bool keep_assign, int* grid_out, hipStream_t s) {
    constexpr int WAVES = 4;
    const int64_t nbatches = cdiv(g.N, 32), wgs = (int64_t)device_cu_count() * (DCH == 4 && g.d <= 40 ? 2 : stream_per_cu(DCH, ASSIGN));
    int64_t G = cdiv(wgs, g.B);
    G = std::min<int64_t>(G, g.fused_grid_cap);
    G = std::min<int64_t>(G, cdiv(nbatches, WAVES));
    const bool runs = !(ASSIGN && DCH == 8) && nbatches > G * WAVES * kStreamRun;
    // (no more of those than run at once)
    if (runs) G = std::min<int64_t>(G, wgs / g.B);
    G = std::max<int64_t>(G, 1);
    auto kern = runs ? stream_update_kernel<BF, DCH, WAVES, ASSIGN, !(ASSIGN && DCH == 8)> : stream_update_kernel<BF, DCH, WAVES, ASSIGN, false>;
    // two batch buffers per wave; at the end the waves' tables and counts
    const size_t lds = std::max((size_t)WAVES * 2 * (DCH * 64 + (ASSIGN ? 0 : 16)) * 16, (size_t)WAVES * 32 * (DCH * 16 + 1) * 4);
    // set once per kernel and device: the launch path stays free of runtime calls afterwards
    static PerDeviceInt attr_set[2];
    if (attr_set[runs].get() == 0) {
        FK_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        attr_set[runs].set(1);
    }
    dim3 grid((unsigned)G, g.B), block(WAVES * 64);
    hipLaunchKernelGGL(kern, grid, block, lds, s, (const uint16_t*)X, (const uintx4*)w.c_frag,
                       (const float*)w.c_bias, assign, w.partial, w.wg_counts, g.N, g.d, g.K, keep_assign ? 1 : 0);
    FK_HIP(hipGetLastError());
    *grid_out = (int)G;
    return FK_OK;
}

template <bool ASSIGN>
static fk_status launch_stream_update_d(const Geometry& g, const Workspace& w, const void* X,
                                        int32_t* assign, bool keep_assign, int* grid_out, hipStream_t s) {
    const bool bf = g.t == FK_BF16;
    switch (g.dchunks) {
        case 2: return bf ? launch_stream_update_t<true, 2, ASSIGN>(g, w, X, assign, keep_assign, grid_out, s)
                          : launch_stream_update_t<false, 2, ASSIGN>(g, w, X, assign, keep_assign, grid_out, s);
        case 4: return bf ? launch_stream_update_t<true, 4, ASSIGN>(g, w, X, assign, keep_assign, grid_out, s)
                          : launch_stream_update_t<false, 4, ASSIGN>(g, w, X, assign, keep_assign, grid_out, s);
        case 8: return bf ? launch_stream_update_t<true, 8, ASSIGN>(g, w, X, assign, keep_assign, grid_out, s)
                          : launch_stream_update_t<false, 8, ASSIGN>(g, w, X, assign, keep_assign, grid_out, s);
    }
    set_error("fused update: no kernel for %d feature chunks", g.dchunks);
    return FK_EUNSUPPORTED;
}

fk_status launch_stream_update(const Geometry& g, const Workspace& w, const void* X,
                               int32_t* assign, bool compute_assign, bool keep_assign, int* grid_out,
                               hipStream_t s) {
    if (g.fused_grid_cap <= 0) {
        set_error("fused update: shape not eligible (needs 16-bit storage, K <= 32, d <= 128)");
        return FK_EUNSUPPORTED;
    }
    return compute_assign ? launch_stream_update_d<true>(g, w, X, assign, keep_assign, grid_out, s)
                          : launch_stream_update_d<false>(g, w, X, assign, keep_assign, grid_out, s);
}

}  // namespace fk
