// Small problems in fp32 storage (K <= 64, d <= 128, at most 2^17 points in all): assignment
// (Eq. 2) and the per-cluster sums of Eq. 3 in one pass over X, without sort or gather.  At
// this size an iteration of the general path is six dependent launches of a few microseconds
// each; here it is two.  (For more points the one-point-per-thread assignment kernel followed by
// the sort-inverse update is faster: this kernel gives every wave all 64 points of a batch.)
//
// The table of sums is K x d floats.  A workgroup of four to sixteen waves walks 64-point batches, which it
// copies to LDS in whole lines one batch ahead: every wave then holds the 64 points (one per lane,
// features in registers) and measures them against its share of the centroid rows by direct
// differences in fp32, exactly as the stand-alone fp32 assignment kernels do (so the assignments
// are bit-identical to theirs); the centroid rows are wave-uniform and come through the scalar
// cache straight into the instructions.  The waves' candidates of a point are merged through LDS
// (smaller distance, then lower index).  Cluster k belongs to wave k % WAVES: that wave alone adds the
// batch's points of its clusters, in index order, to the cluster's row of a K x d table in LDS
// (lane = feature; LDS executes a wave's operations in order, so consecutive points of one cluster
// need no wait beyond the data dependency).  One owner per cluster row and a fixed order: no
// atomics, reproducible sums.  Every workgroup leaves one partial table and one count per cluster;
// the ordinary merge/normalise kernel adds them in workgroup order.
//
// What bounds it at one batch per compute unit (N = 16384): a chain of latencies -- points to LDS,
// 2 x 64 vector instructions per centroid, hand-over, adds.  An iteration takes 16.5 us with it (d = K =
// 64; 28 with four waves that each read all points from memory and the centroids from LDS).
#include <algorithm>

#include "fk_common.h"
#include "fk_device.h"

namespace fk {

constexpr int kF32FusedMaxK = 64;

// LDS, in floats: points [64][DMAX + 4] (four floats of padding: the lanes' 16-byte reads of 64 rows
// then spread over all banks) | table [kF32FusedMaxK][DMAX] | candidates 2 x [WAVES][64] | counts
template <int DMAX, int WAVES>
constexpr size_t f32_fused_lds() {
    return ((size_t)64 * (DMAX + 4) + kF32FusedMaxK * DMAX + 2 * WAVES * 64 + kF32FusedMaxK) * 4;
}

// Grid (G, B): workgroup g handles the 64-point batches g, g + G, ...
// partial: [B][K][G][d] floats, wg_counts: [B][K][G].
// TAIL: rows whose length is no multiple of 16 (a test at every piece of a row cost all others 5 to 14%).
template <int DMAX, int WAVES, bool TAIL>
__global__ __launch_bounds__(WAVES * 64) void f32_update_kernel(
    const float* __restrict__ X, const float* __restrict__ C, int32_t* __restrict__ assign,
    float* __restrict__ partial, int32_t* __restrict__ wg_counts, int64_t N, int d, int len, int K) {
    constexpr int kThreads = WAVES * 64;
    constexpr int NR = DMAX > 64 ? 2 : 1;              // table elements per cluster and lane
    constexpr int LD = DMAX + 4;                       // row stride of the batch in LDS
    constexpr int kPieces = 64 * DMAX / 4 / kThreads;  // 16-byte pieces of a batch per thread
    extern __shared__ float lds_f32[];
    float* xs = lds_f32;
    float* tab = xs + 64 * LD;
    float* cand_d = tab + kF32FusedMaxK * DMAX;
    int* cand_k = (int*)(cand_d + WAVES * 64);
    int* tcnt = cand_k + WAVES * 64;

    const int b = blockIdx.y, G = gridDim.x, wg = blockIdx.x;
    X += (size_t)b * N * len;
    C += (size_t)b * K * len;
    assign += (size_t)b * N;
    const int tid = threadIdx.x, lane = tid & 63;
    const int q = __builtin_amdgcn_readfirstlane(tid >> 6);

    const int64_t nbatches = (N + 63) / 64;
    // this thread's pieces of a batch: consecutive threads take consecutive pieces of a row
    floatx4 ahead[kPieces];
    auto request = [&](int64_t t) {
#pragma unroll
        for (int i = 0; i < kPieces; ++i) {
            const int o = tid + i * kThreads, r = o / (DMAX / 4), j = (o % (DMAX / 4)) * 4;
            ahead[i] = floatx4{0.f, 0.f, 0.f, 0.f};
            if (t * 64 + r < N && j < len) ahead[i] = raw_piece32(X + (size_t)(t * 64 + r) * len, j, len);
        }
    };
    request(wg);
    for (int o = tid; o < K * DMAX; o += kThreads) tab[o] = 0.f;
    if (tid < kF32FusedMaxK) tcnt[tid] = 0;

    for (int64_t t = wg; t < nbatches; t += G) {
        const int64_t base = t * 64;
        const int rows = (int)min((int64_t)64, N - base);
        __syncthreads();                               // the previous batch's readers are done
        if (len & 3) {
#pragma unroll
            for (int i = 0; i < kPieces; ++i) {
                const int j = (tid + i * kThreads) % (DMAX / 4) * 4;
                if (j < len) ahead[i] = settle32(ahead[i], j, len);
            }
        }
#pragma unroll
        for (int i = 0; i < kPieces; ++i) {
            const int o = tid + i * kThreads;
            *(floatx4*)(xs + o / (DMAX / 4) * LD + o % (DMAX / 4) * 4) = ahead[i];
        }
        __syncthreads();
        if (t + G < nbatches) request(t + G);          // lands while this batch is processed
        float x[DMAX];                                 // lane = point
#pragma unroll
        for (int j = 0; j < DMAX; j += 4) {
            const floatx4 v = *(const floatx4*)(xs + lane * LD + j);
            x[j] = v[0]; x[j + 1] = v[1]; x[j + 2] = v[2]; x[j + 3] = v[3];
        }
        float m = INFINITY;
        int a = 0x7FFFFFFF;
        // rows q, q + WAVES, ... ascending with strict '<'; two rows at a time so that the two
        // dependent chains of adds overlap (each row's own sum keeps its order)
        for (int r = q; r < K; r += 2 * WAVES) {
            const int r1 = r + WAVES < K ? r + WAVES : r;   // past the end: row r again (loses the '<')
            const float* c0 = C + (size_t)r * len;
            const float* c1 = C + (size_t)r1 * len;
            float D0 = 0.f, D1 = 0.f;
#pragma unroll
            for (int j = 0; j < DMAX; j += 16) {
                if (j + 16 <= len) {
                    float p[16], q1[16];
#pragma unroll
                    for (int e = 0; e < 16; ++e) { p[e] = c0[j + e]; q1[e] = c1[j + e]; }
                    __builtin_amdgcn_sched_barrier(0);      // both rows asked for before the first wait
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const float u = x[j + e] - p[e], v = x[j + e] - q1[e];
                        D0 = fmaf(u, u, D0);
                        D1 = fmaf(v, v, D1);
                    }
                }
            }
            if constexpr (TAIL) {
                // the last len % 16 features, from LDS: once in the code, wherever the row ends
                int j = len & ~15;
                const float* xt = xs + lane * LD;
                if (len & 8) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float t = xt[j + e], u = t - c0[j + e], v = t - c1[j + e];
                        D0 = fmaf(u, u, D0);
                        D1 = fmaf(v, v, D1);
                    }
                    j += 8;
                }
                for (; j < len; ++j) {
                    const float t = xt[j], u = t - c0[j], v = t - c1[j];
                    D0 = fmaf(u, u, D0);
                    D1 = fmaf(v, v, D1);
                }
            }
            if (D0 < m) { m = D0; a = r; }
            if (D1 < m) { m = D1; a = r1; }
        }
        cand_d[q * 64 + lane] = m;
        cand_k[q * 64 + lane] = a;
        __syncthreads();
        // every wave merges for itself: lane = point
        float bm = cand_d[lane];
        int bk = cand_k[lane];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) {
            const float dm = cand_d[w * 64 + lane];
            const int dk = cand_k[w * 64 + lane];
            if (dm < bm || (dm == bm && dk < bk)) { bm = dm; bk = dk; }
        }
        bk = min(bk, K - 1);   // only reachable with non-finite input; keeps the index in range
        const bool valid = lane < rows;
        if (q == 0 && valid) assign[base + lane] = bk;

        // the batch's points of this wave's clusters, in index order
        uint64_t mine = __ballot(valid && (bk & (WAVES - 1)) == q);
        while (mine) {
            const int p = __builtin_ctzll(mine);
            mine &= mine - 1;
            const int k = __builtin_amdgcn_readlane(bk, p);
            float* trow = tab + k * DMAX;
#pragma unroll
            for (int u = 0; u < NR; ++u) {
                const int j = lane + 64 * u;
                if (j < d) trow[j] += xs[p * LD + j];
            }
            if (lane == 0) tcnt[k] += 1;
        }
    }

    // the owner of a row wrote it: no barrier needed before reading it back
    for (int k = q; k < K; k += WAVES) {
        float* row = partial + (((size_t)b * K + k) * G + wg) * d;
#pragma unroll
        for (int u = 0; u < NR; ++u) {
            const int j = lane + 64 * u;
            if (j < d) row[j] = tab[k * DMAX + j];
        }
        if (lane == 0) wg_counts[((size_t)b * K + k) * G + wg] = tcnt[k];
    }
}

// ------------------------------------------------------------------------------------
template <int DMAX, int WAVES, bool TAIL>
static fk_status launch_f32_update_r(const Geometry& g, const Workspace& w, const float* X,
                                     const float* C, int32_t* assign, int* grid_out,
                                     hipStream_t s) {
    auto kern = f32_update_kernel<DMAX, WAVES, TAIL>;
    const size_t lds = f32_fused_lds<DMAX, WAVES>();
    // set / queried once per kernel and device: the launch path stays free of runtime queries afterwards
    static PerDeviceInt per_cu;
    if (per_cu.get() == 0) {
        FK_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        int q = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&q, kern, WAVES * 64, lds) != hipSuccess || q < 1) q = 1;
        per_cu.set(q);
    }
    // (a fourth workgroup of eight waves only adds tables to merge: N = 60000, d = 32, K = 64, six iterations:
    // 150 us with, 135 without)
    int64_t G = cdiv((int64_t)device_cu_count() * (WAVES == 4 ? per_cu.get() : std::min(per_cu.get(), 3)), g.B);
    G = std::min<int64_t>(G, g.f32_grid_cap);
    G = std::min<int64_t>(G, cdiv(g.N, 64));
    G = std::max<int64_t>(G, 1);
    G = cdiv(cdiv(g.N, 64), cdiv(cdiv(g.N, 64), G));   // no more tables than as many rounds need: 7 x 13000, d = 128, K = 64 636 -> 518
    dim3 grid((unsigned)G, g.B), block(WAVES * 64);
    hipLaunchKernelGGL(kern, grid, block, lds, s, X, C, assign, w.partial, w.wg_counts, g.N, g.d, g.len, g.K);
    FK_HIP(hipGetLastError());
    *grid_out = (int)G;
    return FK_OK;
}

template <int DMAX, int WAVES>
static fk_status launch_f32_update_t(const Geometry& g, const Workspace& w, const float* X, const float* C, int32_t* assign,
                                     int* grid_out, hipStream_t s) {
    return g.len % 16 == 0 ? launch_f32_update_r<DMAX, WAVES, false>(g, w, X, C, assign, grid_out, s)
                           : launch_f32_update_r<DMAX, WAVES, true>(g, w, X, C, assign, grid_out, s);
}

fk_status launch_f32_update(const Geometry& g, const Workspace& w, const void* X,
                            const float* C_f32, int32_t* assign, int* grid_out, hipStream_t s) {
    if (g.f32_grid_cap <= 0) {
        set_error("fused fp32 update: shape not eligible (fp32 storage, K <= 64, d <= 128, few points)");
        return FK_EUNSUPPORTED;
    }
    const float* Xf = (const float*)X;
    // Waves per workgroup.  Few clusters leave more waves without rows, and smaller workgroups are more of
    // them, each with its own chain of additions (six iterations, us, 4 / 8 / 16 waves, before the rows came
    // in pairs of loads):
    //   N = 16384, d = 64:    K = 4 86 / 91 / 99, K = 8 88 / 82 / 91, K = 32 122 / 97 / 95, K = 64 164 / 124 / 111
    //   N = 2^17,  d = 64:    K = 8 165 / 185, K = 16 185 / 185, K = 64 300 / 284
    //   N = 2^17,  d = 128:   K = 8 285 / 351, K = 16 335 / 356, K = 64 630 / 659;  N = 60000: K = 64 407 / 391
    //   N = 7 x 13000, d = 128: K = 8 254 / 417, K = 64 638 / 792
    const bool once = cdiv(g.N, 64) * g.B <= device_cu_count();      // up to one batch per compute unit
    const bool four = g.K <= 4 || (!once && (g.K <= 8 || g.d > 64));
    if (g.d <= 32)
        return four ? launch_f32_update_t<32, 4>(g, w, Xf, C_f32, assign, grid_out, s)
                    : launch_f32_update_t<32, 8>(g, w, Xf, C_f32, assign, grid_out, s);
    if (g.d > 64)
        return four ? launch_f32_update_t<128, 4>(g, w, Xf, C_f32, assign, grid_out, s)
                    : launch_f32_update_t<128, 8>(g, w, Xf, C_f32, assign, grid_out, s);
    if (four) return launch_f32_update_t<64, 4>(g, w, Xf, C_f32, assign, grid_out, s);
    if (once && g.K > 16) return launch_f32_update_t<64, 16>(g, w, Xf, C_f32, assign, grid_out, s);
    return launch_f32_update_t<64, 8>(g, w, Xf, C_f32, assign, grid_out, s);
}

}  // namespace fk
