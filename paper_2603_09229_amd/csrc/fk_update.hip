// Segment-level aggregation and normalisation of the sort-inverse update (paper Section
// 4.2, Algorithm 3; Eq. 3).
//
// The paper cuts the sorted order into fixed chunks, accumulates each cluster-id segment
// of a chunk on chip and merges it with one atomic_add per segment.  Here the cut follows
// the segments instead: cluster k's run of n_k sorted positions is split into
// ceil(n_k / R) "items" of at most R positions, one wave reduces one item in registers and
// writes one partial row, and a second kernel adds a cluster's partial rows in item order.
// That keeps the paper's bound on merges (at most K + N/R rows are merged) but needs no
// atomics at all and is bit-reproducible.  X is gathered by whole rows through sorted_idx
// and never permuted in memory.
#include "fk_common.h"
#include "fk_device.h"

namespace fk {

namespace {

// Points per item of a cluster of n, a multiple of R; the item table has room for ceil(n / R) of them.  A wave
// adds an item's points and one workgroup merges the cluster's items, `balance` rows in the time of one point: beyond
// sqrt(balance n) items the merge costs more than their shorter chains give.  fk_update with clusters of Zipf
// sizes, us, items of R points / this: 154912 points, d = 80, K = 649 108 / 54; 2^23, d = 128, K = 4096 726 / 628 (the merge
// alone 194 before); fp32 88476, d = 104, K = 660 76 / 54.
// Most clusters are shorter than that and skip the divisions and the root, which cost 61312 merges of two rows each 12%
// (16 instances of 7440 fp32 points, d = 134, K = 3832 165 us with them, 150 without).
__device__ __forceinline__ int item_length(int n, int R, float balance) {
    if (n <= 64 * R) return R;
    const int items = (n + R - 1) / R, most = max(64, (int)sqrtf(balance * (float)n));
    return items <= most ? R : (items + most - 1) / most * R;
}

// Largest k in [0,K) with item_off[k] <= item, found by the whole wave 64 probes at a
// time.  Requires item < item_off[K]; the cluster found is then non-empty.
__device__ __forceinline__ int find_cluster(const int32_t* __restrict__ item_off, int K,
                                            int item, int lane) {
    int lo = 0, hi = K;
    while (hi - lo > 1) {
        const int step = (hi - lo + 63) >> 6;
        const int probe = lo + lane * step;
        const bool le = probe < hi && item_off[probe] <= item;
        const int cnt = __popcll(__ballot(le));   // monotone: a prefix of the lanes
        lo += (cnt - 1) * step;
        hi = min(hi, lo + step);
    }
    return lo;
}

// Adds the rows' pieces of a batch of loads to the lane's sums, in pairs first: a large cluster's items are hundreds of
// rows long, and so are a wave's shares of one in gather_update_kernel.  With every row a link of one chain the means of
// 300000 points in one cluster (fp32, d = 96, K = 400: items of 384 rows) were 2.6e-7 off, with items of 128 2.1e-7; in pairs
// 1.5e-7, in the same time.
template <int EPL, bool BF, int U>
__device__ __forceinline__ void add_in_pairs(const uintx4 (&v)[U], float (&acc)[EPL]) {
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
        float t[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if constexpr (EPL == 4) t[u] = __uint_as_float(v[u][e]);
            else t[u] = lp_to_float((uint16_t)(e & 1 ? v[u][e / 2] >> 16 : v[u][e / 2] & 0xFFFFu), BF);
        }
#pragma unroll
        for (int half = U / 2; half > 0; half /= 2)
#pragma unroll
            for (int u = 0; u < half; ++u) t[u] += t[u + half];
        acc[e] += t[0];
    }
}

}  // namespace

// WPI waves per item (1, or all 4 of the workgroup for the long items of few-cluster
// shapes).  EPL elements of 16 bytes per lane (8 for 16-bit types, 4 for fp32); 2^lpr_log2
// lanes span a row, so a wave reads 64 >> lpr_log2 rows per load instruction.  With WPI = 4
// wave w takes the 64-row batches w, w+4, ... of the item and the four wave sums are added in
// wave order through LDS.
// RAGGED: rows whose length is no multiple of 8, read as they are stored (skipped at run time, that code costs
// the others 3%: 342180 points, d = 512, K = 34: 68.3 -> 70.4 us).
// ONCE: loads that ask for no place in the caches, see reads_once.
template <int EPL, bool BF, int WPI, bool RAGGED, bool ONCE>
__global__ __launch_bounds__(256) void segment_reduce_kernel(
    const void* __restrict__ Xv, const int32_t* __restrict__ sorted_idx,
    const int32_t* __restrict__ seg_off, const int32_t* __restrict__ item_off,
    float* __restrict__ partial, int64_t N, int d, int K, int R, int64_t max_items,
    int lpr_log2, int row_len, float balance) {
    const int len = RAGGED ? row_len : d;
    __shared__ float wsum[WPI == 4 ? 4 : 1][WPI == 4 ? 512 : 1];
    const int b = blockIdx.y;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t item = WPI == 4 ? (int64_t)blockIdx.x : (int64_t)blockIdx.x * 4 + wave;
    const int part = WPI == 4 ? wave : 0;          // which share of the item this wave takes
    seg_off += (size_t)b * (K + 1);
    item_off += (size_t)b * (K + 1);
    sorted_idx += (size_t)b * N;
    if (item >= item_off[K]) return;   // uniform over the waves that share an item
    const int k = find_cluster(item_off, K, (int)item, lane);
    const int first_pos = seg_off[k], n = seg_off[k + 1] - first_pos, length = item_length(n, R, balance);
    const int64_t offset = (int64_t)((int)item - item_off[k]) * length;
    if (offset >= n) return;           // (uniform likewise)
    const int start = first_pos + (int)offset, end = first_pos + (int)min((int64_t)n, offset + length);

    const int LPR = 1 << lpr_log2, S = 64 >> lpr_log2;
    const int slot = lane >> lpr_log2;
    const char* X = (const char*)Xv + (size_t)b * N * len * (16 / EPL);
    // rows wider than one wave-load (64 lanes x 16 bytes) are reduced one column block at a time
    const int ncb = (d + 64 * EPL - 1) / (64 * EPL);
    for (int cb = 0; cb < ncb; ++cb) {
        const int col = cb * 64 * EPL + (lane & (LPR - 1)) * EPL;
        const bool active = col < d;
        // this lane's piece of a row, or where that would cross the row's end the one that ends
        // there; of the sums only those at its own columns are kept (from len on nobody reads them)
        const int first = RAGGED ? min(col, len - EPL) : col;
        const char* mine = X + first * (16 / EPL);
        const int row_bytes = len * (16 / EPL);
        float acc[EPL];
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[e] = 0.f;

        constexpr int U = 8;
        for (int r0 = start + part * 64; r0 < end; r0 += 64 * WPI) {
            const int nrows = min(64, end - r0);
            const int myidx = lane < nrows ? sorted_idx[r0 + lane] : 0;
            for (int q = 0; q < nrows; q += S * U) {
                uintx4 v[U];
                bool ok[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int rr = q + u * S + slot;
                    const int idx = __shfl(myidx, rr & 63);
                    ok[u] = active && rr < nrows;
                    v[u] = uintx4{0u, 0u, 0u, 0u};
                    if (ok[u]) {
                        const char* at = mine + (int64_t)idx * row_bytes;
                        if constexpr (ONCE) v[u] = __builtin_nontemporal_load((const uintx4*)at);
                        else v[u] = RAGGED ? (uintx4)*(const uintx4_any*)at : *(const uintx4*)at;
                    }
                }
                add_in_pairs<EPL, BF>(v, acc);
            }
        }
        // add the row slots of the wave together (fixed butterfly order)
        for (int o = LPR; o < 64; o <<= 1) {
#pragma unroll
            for (int e = 0; e < EPL; ++e) acc[e] += __shfl_xor(acc[e], o);
        }
        if (slot == 0 && active) {
            if (WPI == 1) {
                float* out = partial + ((size_t)b * max_items + item) * d + first;
                if (!RAGGED || first == col) {
#pragma unroll
                    for (int e = 0; e < EPL; e += 4)
                        *(floatx4*)(out + e) = floatx4{acc[e], acc[e + 1], acc[e + 2], acc[e + 3]};
                } else {
#pragma unroll
                    for (int e = 0; e < EPL; ++e)
                        if (first + e >= col) out[e] = acc[e];
                }
            } else {
#pragma unroll
                for (int e = 0; e < EPL; ++e)
                    if (!RAGGED || first + e >= col) wsum[wave][first + e] = acc[e];
            }
        }
    }
    if (WPI == 4) {
        __syncthreads();
        for (int j = threadIdx.x; j < d; j += 256) {
            const float s = ((wsum[0][j] + wsum[1][j]) + wsum[2][j]) + wsum[3][j];
            partial[((size_t)b * max_items + item) * d + j] = s;
        }
    }
}

// Where a cluster's mean goes, and what is added to its sum on the way.
struct EmitTo {
    const float* C_prev;
    float* C_out;
    uint16_t* C_lp_out;
    float* C_lp_f32_out;
    uint16_t* c_frag;
    float* c_bias;
    int32_t* counts;
    float* sums;
    const float* late_sums;
    const int32_t* late_counts;
    int d, K, B, ktiles, dch, accumulate, normalise, bf, late, row_len;
    // fp32: the split centroids of the filtered assignment (fk_f32_filter.hip) with the shift that the first
    // assignment of the call has left, c2 their norms; the lengths of its lists, which the next assignment starts from
    uint16_t* c_split;
    const float* shift;
    float* c2;
    int32_t *list_len, *pair_len;
};

// Row k of the split centroids, from its shifted values in `row` (d floats of LDS, not yet behind a barrier): what
// f32_split_layout_kernel writes for it, so that the next assignment of the call needs no launch of that kernel (5 to 8 us).  Rows beyond
// K and features beyond d keep what that kernel's launch in the first assignment wrote there, and so does the shift, a mean of
// points: the bound grows with the squared distances from it of points and centroids.  With a mean of the starting centroids instead a start
// away from the points left every point open in every iteration; laid out anew in the second and every eighth iteration it cost 4 to 6 us
// a launch.  300000 normally distributed points, d = 96, K = 400, ten iterations from rows of theirs, us, mean of the starting centroids / of
// points: 1435 / 1434; one feature of the start 300 off 10938 / 1597, 30 off 2043 / 1417, every feature 10 off 5862 / 1518; one row in 997 a thousand
// times as long 13338 / 1370.
__device__ __forceinline__ void emit_split(const EmitTo& to, int b, int k, const float* row, bool odd) {
    const int tid = threadIdx.x, d = to.d, T = (int)blockDim.x;
    __shared__ int fits;
    uint16_t* tile = to.c_split + ((size_t)b * to.ktiles + (k >> 5)) * (2 * to.dch + 1) * 512;
    const int never = __syncthreads_or(odd);
    if (tid < 64) {
        double n2 = 0.0;
        for (int j = tid; j < d; j += 64) n2 += (double)row[j] * (double)row[j];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) n2 += __shfl_xor(n2, o);
        if (tid == 0) {
            float norm;
            *(uintx4*)(tile + (2 * to.dch * 64 + (k & 31)) * 8) = split_bias(n2, to.dch * 16, never != 0, &norm);
            to.c2[(size_t)b * to.ktiles * 32 + k] = norm;
            fits = !never && n2 < 1e38;
            if (k == 0) { to.list_len[b] = 0; to.pair_len[b] = 0; }
        }
    }
    __syncthreads();
    for (int j = tid; j < d; j += T) {
        const float v = fits ? row[j] : 0.f;
        const uint16_t hi = float_to_lp(v, true), lo = float_to_lp(v - lp_to_float(hi, true), true);
        uint16_t* at = tile + (2 * (j >> 4) * 64 + (((j >> 3) & 1) << 5) + (k & 31)) * 8 + (j & 7);
        at[0] = hi;
        at[512] = lo;
    }
}

// The end of an update, by the whole workgroup: cluster k of instance b has n points (late ones not among
// them yet), sum_of(j) is the sum of their feature j.  Optionally added onto sums/counts already stored
// (chunked mode; kLate: followed by the parts that have waited for their turn), optionally
// normalised into centroids (Algorithm 3, last loop; an empty cluster keeps its previous
// centroid).  When c_frag is given, the rounded centroid is also
// written in MFMA fragment order together with its score bias -||c||^2/2, so the next
// assignment needs no separate re-layout pass; kSplit: so are fp32 ones (emit_split).  nrm: d floats of LDS.
template <bool kLate, bool RAGGED, bool kSplit, class Sum>
__device__ __forceinline__ void emit_centroid(const EmitTo& to, int b, int k, int n, float* nrm, Sum sum_of) {
    const int tid = threadIdx.x, d = to.d, K = to.K, T = (int)blockDim.x;
    const int len = RAGGED ? to.row_len : d;
    if constexpr (kLate)
        for (int q = 0; q < to.late; ++q) n += to.late_counts[((size_t)q * to.B + b) * K + k];
    bool odd = false;
    for (int j = tid; j < d; j += T) {
        float s = sum_of(j);
        const size_t o = ((size_t)b * K + k) * d + j;
        if (to.accumulate) s += to.sums[o];
        if constexpr (kLate)
            for (int q = 0; q < to.late; ++q) s += to.late_sums[(size_t)q * to.B * K * d + o];
        if (to.sums) to.sums[o] = s;
        if (to.normalise) {
            // the caller's rows have no padding; past their end everything is zero
            const size_t at = ((size_t)b * K + k) * len + j;
            const float c = RAGGED && j >= len ? 0.f : n > 0 ? (float)((double)s / (double)n) : to.C_prev[at];
            const uint16_t lp = float_to_lp(c, to.bf);
            if (!RAGGED || j < len) {
                to.C_out[at] = c;
                if (to.C_lp_out) to.C_lp_out[at] = lp;
                if (to.C_lp_f32_out) to.C_lp_f32_out[at] = c;
            }
            if (to.c_frag) {
                // fragment order: tile k/32, chunk j/16, lane (j%16)/8*32 + k%32, element j%8
                const size_t pos = ((((size_t)b * to.ktiles + (k >> 5)) * to.dch + (j >> 4)) * 64 +
                                    (((j >> 3) & 1) << 5) + (k & 31)) * 8 + (j & 7);
                to.c_frag[pos] = lp;
                const float f = lp_to_float(lp, to.bf);
                nrm[j] = __fmul_rn(f, f);
            }
            if (kSplit && to.c_split) {
                nrm[j] = j < len ? c - to.shift[(size_t)b * to.dch * 16 + j] : 0.f;
                odd |= !(fabsf(c) < INFINITY);
            }
        }
    }
    if (tid == 0) to.counts[(size_t)b * K + k] = n;
    if (to.normalise && to.c_frag) {
        __syncthreads();
        // same association as the stand-alone layout kernel: groups of 8 features first (one
        // thread per group; the first wave holds them all, d <= 512), then the groups in order
        if (tid < 64) {
            float ss = 0.f;
            if (tid * 8 < d) {
                for (int e = 0; e < 8; ++e) ss = __fadd_rn(ss, nrm[tid * 8 + e]);
            }
            float n2 = 0.f;
            for (int g0 = 0; g0 * 8 < d; ++g0)
                n2 = __fadd_rn(n2, __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(ss), g0)));
            if (tid == 0) to.c_bias[((size_t)b * to.ktiles) * 32 + k] = -0.5f * n2;
        }
    }
    if (kSplit && to.c_split) emit_split(to, b, k, nrm, odd);
}

// One workgroup (256 threads, or 1024 when clusters have many items) per cluster: s_k = sum
// of the cluster's item rows in a fixed order, n_k = seg_off[k+1] - seg_off[k]; then emit_centroid.
// kSplit: with the code for split centroids, which costs the others time where it is only skipped (32 instances of 3000 points,
// d = 40, K = 100: 9.2 -> 10.5 us).
template <bool kLate, bool RAGGED, bool kSplit>
__global__ __launch_bounds__(1024) void finalize_kernel(
    const float* __restrict__ partial, const int32_t* __restrict__ seg_off,
    const int32_t* __restrict__ item_off, EmitTo to, int R, float balance, int64_t max_items,
    const int32_t* __restrict__ wg_counts, int G) {
    // dynamic LDS: 4 floats per thread for the row sums, then d floats for the squared entries
    // (a fixed worst-case array would cap the small workgroups of many-cluster shapes at a
    // few per CU)
    const int d = to.d, K = to.K;
    extern __shared__ float fin_lds[];
    float* red = fin_lds;
    float* nrm = fin_lds + 4 * blockDim.x;
    __shared__ int cred[16];
    const int b = blockIdx.y, k = blockIdx.x, tid = threadIdx.x;
    int dpow = 4;
    while (dpow < d) dpow <<= 1;
    const int LR = dpow >> 2;                     // threads per row, 4 features each
    const int slots = (int)blockDim.x / LR, slot = tid / LR, col = (tid % LR) * 4;
    int i0, i1;
    if (wg_counts) {
        // few-cluster path: cluster k owns G partial rows and G partial counts
        i0 = k * G;
        i1 = i0 + G;
        int v = 0;
        for (int g = tid; g < G; g += (int)blockDim.x) v += wg_counts[((size_t)b * K + k) * G + g];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
        if ((tid & 63) == 0) cred[tid >> 6] = v;
    } else {
        seg_off += (size_t)b * (K + 1);
        item_off += (size_t)b * (K + 1);
        i0 = item_off[k];
        const int n = seg_off[k + 1] - seg_off[k], length = item_length(n, R, balance);
        i1 = length == R ? item_off[k + 1] : i0 + (n + length - 1) / length;
    }
    // read the running count before anyone overwrites it (barrier below)
    const int n_prev = to.accumulate ? to.counts[(size_t)b * K + k] : 0;
    const float* P = partial + (size_t)b * max_items * d;
    // eight rows in flight per thread; the eight running sums are added in a fixed order
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    if (col < d) {
        floatx4 a8[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) a8[u] = floatx4{0.f, 0.f, 0.f, 0.f};
        for (int it = i0 + slot; it < i1; it += 8 * slots) {
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int r = it + u * slots;
                if (r < i1) a8[u] += *(const floatx4*)(P + (size_t)r * d + col);
            }
        }
        acc = ((a8[0] + a8[1]) + (a8[2] + a8[3])) + ((a8[4] + a8[5]) + (a8[6] + a8[7]));
    }
    // rows of one wave first (fixed butterfly order), then the waves' sums through LDS: with a row
    // of 64 features 16 partial sums are added one after the other at the end instead of 64.  (A
    // workgroup of one wave has few rows to add: 532760 clusters of d = 32, most of them empty, 206 us with
    // the exchange, 185 without.)
    const bool by_wave = LR < 64 && blockDim.x > 64;
    if (by_wave)
        for (int o = LR; o < 64; o <<= 1) {
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] += __shfl_xor(acc[e], o);
        }
    const int sums_left = by_wave ? (int)blockDim.x >> 6 : slots;
    if (!by_wave) *(floatx4*)&red[slot * dpow + col] = acc;
    else if ((tid & 63) < LR) *(floatx4*)&red[(tid >> 6) * dpow + col] = acc;
    __syncthreads();
    int n = n_prev;
    if (wg_counts) {
        for (int q = 0; q < ((int)blockDim.x + 63) / 64; ++q) n += cred[q];
    } else {
        n += seg_off[k + 1] - seg_off[k];
    }
    emit_centroid<kLate, RAGGED, kSplit>(to, b, k, n, nrm, [&](int j) {
        float s = 0.f;
        for (int q = 0; q < sums_left; ++q) s += red[q * dpow + j];   // fixed order
        return s;
    });
}

// ------------------------------------------------------------------------------------
// Small instances (choose_gather_parts): the whole update, or all of it but the merge, in one launch and without a sort.  A workgroup
// owns one cluster (or, with G parts, the points of one cluster in a G-th of the instance), reads every
// assignment of its part, keeps the indices of its own points and adds their rows.  Every workgroup reads
// all assignments, K*N in all, which come from L2; what it saves are the four to seven dependent
// launches of the sort, each bound by latency at this size.
// Wave w takes the 256-key blocks w, w + WAVES, ...; its matches collect in a list of its own in LDS and are
// added a group of rows at a time, with the row pieces per lane of segment_reduce_kernel, where every wave has several
// blocks, otherwise after all waves have shared them out evenly.  Which wave adds a row and in which place follows from
// the assignments alone: fixed order, no atomics.
// A compute unit's instructions bound a large cluster, so whole batches of rows are loaded without a test for each:
// all points in one cluster, us, with tests and without: 2010 fp32, d = 256, K = 467 27.1 -> 18.9; 4096, d = 256, K = 500 33.2 ->
// 20.8 (twice the loads in flight: 32.2).  Shares of few blocks: 1024 fp32, d = 512, K = 20, where one wave had a
// block's 256 rows, 51.4 -> 12.7 with both.
template <int EPL, bool BF, bool RAGGED, int WAVES>
__global__ __launch_bounds__(WAVES * 64) void gather_update_kernel(
    const void* __restrict__ Xv, const int32_t* __restrict__ keys, EmitTo to,
    float* __restrict__ partial, int32_t* __restrict__ wg_counts, int64_t N, int G, int merged, int lpr_log2) {
    constexpr int kBlocks = EPL == 4 ? 2 : 1;      // column blocks of 64 lanes x 16 bytes in the widest row
    constexpr int kAhead = 4;                      // key loads in flight per wave
    constexpr int kLoads = 8;                      // row loads in flight per lane
    constexpr int kHold = 256, kList = kHold + 256; // waiting + one block's matches
    typedef int32_t intx4_any __attribute__((ext_vector_type(4), aligned(4)));
    __shared__ int list[WAVES][kList];
    __shared__ int pool[WAVES * kHold];
    __shared__ float nrm[512];                     // squared entries
    __shared__ int left[WAVES], cred[WAVES];
    const int d = to.d, K = to.K, len = RAGGED ? to.row_len : d;
    const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // Workgroups go to the eight XCDs in turn.  With a multiple of eight of them in an instance a cluster that is large in all
    // instances would be added by one XCD alone, so the clusters change places from instance to instance (from every 8 / apart
    // to the next).  The middle one with all points, us, sorted / in place / moved: 50 instances of 4000 fp32 points, d = 64, K = 8
    // 23 / 44 / 25; 32 x 8000, d = 128, K = 8 32 / 54 / 29; 128 x 1000 fp32, d = 256, K = 4 35 / 56 / 28; 4 x 4000 fp32, d = 256, K = 60
    // 26 / 28 / 23.  Odd numbers spread by themselves, and moving cost 100 x 4000 fp32, d = 128, K = 3 36 -> 53.
    const int turn = blockIdx.x / G, part = blockIdx.x - turn * G;
    const int apart = min((int)gridDim.x & -(int)gridDim.x, 8);
    int k = turn;
    if (apart > 1 && b * apart > 7) k = (int)((uint32_t)(turn + (b * apart >> 3)) % (uint32_t)K);
    const int64_t share = (N + G - 1) / G;
    const int lo = (int)min(N, part * share), hi = (int)min(N, lo + share);
    keys += (size_t)b * N;
    const int n_prev = to.accumulate ? to.counts[(size_t)b * K + k] : 0;
    // ids out of range belong to the first and the last cluster
    const int32_t k_lo = k == 0 ? INT32_MIN : k, k_hi = k == K - 1 ? INT32_MAX : k;
    const uint32_t span = (uint32_t)k_hi - (uint32_t)k_lo;

    const int LPR = 1 << lpr_log2, S = 64 >> lpr_log2, slot = lane >> lpr_log2;
    const int row_bytes = len * (16 / EPL);
    const char* X = (const char*)Xv + (size_t)b * N * row_bytes;
    float acc[kBlocks][EPL];
#pragma unroll
    for (int cb = 0; cb < kBlocks; ++cb)
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[cb][e] = 0.f;
    int* mylist = list[wave];
    const int group = min(max(64, kLoads * S), kHold), hold = hi - lo >= 4 * WAVES * 256 ? group : kHold;
    int held = 0, own = 0;

    auto add_rows = [&](const int* rows, int count) {
        constexpr int U = kLoads;
#pragma unroll
        for (int cb = 0; cb < kBlocks; ++cb) {
            const int col = cb * 64 * EPL + (lane & (LPR - 1)) * EPL;
            if (cb > 0 && cb * 64 * EPL >= d) break;
            // where a lane's piece would cross the row's end: the one that ends there (see segment_reduce_kernel); lanes
            // beyond the row read it too, and nobody their sums
            const uint32_t mine = min(col, len - EPL) * (16 / EPL);
            auto piece = [&](int rr) -> uintx4 {
                const char* at = X + (mine + (uint32_t)rows[rr] * (uint32_t)row_bytes);
                return RAGGED ? (uintx4)*(const uintx4_any*)at : *(const uintx4*)at;
            };
            uintx4 v[U];
            int q = slot;
            for (; q - slot + S * U <= count; q += S * U) {
#pragma unroll
                for (int u = 0; u < U; ++u) v[u] = piece(q + u * S);
                add_in_pairs<EPL, BF>(v, acc[cb]);
            }
            if (q - slot < count) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    v[u] = uintx4{0u, 0u, 0u, 0u};
                    if (q + u * S < count) v[u] = piece(q + u * S);
                }
                add_in_pairs<EPL, BF>(v, acc[cb]);
            }
        }
    };

    const uint64_t lt = (1ull << lane) - 1ull;
    // one block's matches (of every key, or only of those before hi) go on the list
    auto take = [&](const intx4_any& kv, int at, bool whole) {
        uint64_t mm[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) mm[e] = __ballot((uint32_t)kv[e] - (uint32_t)k_lo <= span && (whole || at + e < hi));
        if ((mm[0] | mm[1] | mm[2] | mm[3]) == 0) return;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if ((mm[e] >> lane) & 1) mylist[held + __popcll(mm[e] & lt)] = at + e;
            held += __popcll(mm[e]);
        }
        __builtin_amdgcn_wave_barrier();
        while (held > hold) {
            held -= group;
            own += group;
            add_rows(mylist + held, group);
        }
        __builtin_amdgcn_wave_barrier();
    };
    constexpr int kStride = WAVES * 256;
    int base = lo + wave * 256;
    for (; base + (kAhead - 1) * kStride + 256 <= hi; base += kAhead * kStride) {
        intx4_any kv[kAhead];
#pragma unroll
        for (int a = 0; a < kAhead; ++a) kv[a] = *(const intx4_any*)(keys + (base + a * kStride + lane * 4));
#pragma unroll
        for (int a = 0; a < kAhead; ++a) take(kv[a], base + a * kStride + lane * 4, true);
    }
    if (base < hi) {
        intx4_any kv[kAhead];
#pragma unroll
        for (int a = 0; a < kAhead; ++a) {
            const int at = base + a * kStride + lane * 4;
            kv[a] = intx4_any{0, 0, 0, 0};
            if (at + 4 <= hi) {
                kv[a] = *(const intx4_any*)(keys + at);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (at + e < hi) kv[a][e] = keys[at + e];
            }
        }
#pragma unroll
        for (int a = 0; a < kAhead; ++a)
            if (base + a * kStride < hi) take(kv[a], base + a * kStride + lane * 4, false);
    }
    // what is left is shared out again: a part of few blocks may have all its rows on one wave's list, and most
    // clusters here have a few rows in all, which one wave adds in one batch while the others are done
    if (lane == 0) { left[wave] = held; cred[wave] = own + held; }
    __syncthreads();
    int n = n_prev, rest = 0, before = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        n += cred[w];
        before += w < wave ? left[w] : 0;
        rest += left[w];
    }
    for (int i = lane; i < held; i += 64) pool[before + i] = mylist[i];
    __syncthreads();
    const int unit = 8 * S, each = ((rest + WAVES - 1) / WAVES + unit - 1) & -unit;       // (a power of two)
    const int from = wave * each;
    if (from < rest) add_rows(pool + from, min(each, rest - from));
    const bool busy = own > 0 || from < rest;

    constexpr int kRow = kList;                    // (no list is read any more)
    float* red = (float*)&list[0][0];
    if (busy) {
#pragma unroll
        for (int cb = 0; cb < kBlocks; ++cb) {
            if (cb > 0 && cb * 64 * EPL >= d) break;
            const int col = cb * 64 * EPL + (lane & (LPR - 1)) * EPL;
            const int first = RAGGED ? min(col, len - EPL) : col;
            for (int o = LPR; o < 64; o <<= 1) {
#pragma unroll
                for (int e = 0; e < EPL; ++e) acc[cb][e] += __shfl_xor(acc[cb][e], o);
            }
            if (slot == 0 && col < d) {
#pragma unroll
                for (int e = 0; e < EPL; ++e)
                    if (!RAGGED || first + e >= col) red[wave * kRow + first + e] = acc[cb][e];
            }
        }
    }
    if (lane == 0) left[wave] = busy ? 1 : 0;      // (read by everyone before the last barrier)
    __syncthreads();
    auto sum_of = [&](int j) {
        float t[WAVES];                            // (in pairs: a few additions to the largest sums, not one per wave)
#pragma unroll
        for (int w = 0; w < WAVES; ++w) t[w] = left[w] ? red[w * kRow + j] : 0.f;
#pragma unroll
        for (int half = WAVES / 2; half > 0; half /= 2)
#pragma unroll
            for (int w = 0; w < half; ++w) t[w] += t[w + half];
        return t[0];
    };
    if (merged) {                                  // a row and a count for the merge kernel
        const size_t row = ((size_t)b * K + k) * G + part;
        for (int j = tid; j < d; j += WAVES * 64) partial[row * d + j] = sum_of(j);
        if (tid == 0) wg_counts[row] = n - n_prev;
        return;
    }
    emit_centroid<false, RAGGED, EPL == 4>(to, b, k, n, nrm, sum_of);
}

// ------------------------------------------------------------------------------------
static int ceil_log2(int v) {
    int b = 0;
    while ((1 << b) < v) ++b;
    return b;
}

// Threads of a merge workgroup.
static int merge_threads(const Geometry& g) {
    // few clusters with many partial rows each: more rows in flight per workgroup
    // ... and many clusters with few rows each (up to 4, or up to 8 when there are thousands of
    // clusters to spread over the chip): the smallest workgroup that still has a thread per feature
    int threads = g.max_items / g.K > 64 ? 1024 : 256;
    if (g.d <= 128 && (g.max_items / g.K <= 4 || (g.max_items / g.K <= 8 && (int64_t)g.K * g.B >= 4096))) threads = 64;
    return threads;
}

// Rows of four features per thread that a merge workgroup adds at a time, by the rows of 16 bytes per lane that
// the waves of an item do (see item_length).
static float item_balance(const Geometry& g) {
    return (float)merge_threads(g) / (g.t == FK_F32 ? 64.f : 128.f) / (float)g.waves_per_item;
}

// Whether the reduction's loads carry the non-temporal hint: X larger than the last-level cache and rows of
// at least a cache line.  What the caches hold of a smaller X the next pass over it finds there, and a line that two rows share would be
// fetched twice.  us without and with the hint.  fk_update, fp16, K = 500, d = 128: 1.2 million points 84.0 81.3, 1.6 million 115.3 102.7;
// 2^23, K = 4096 535 493 (the reduction 406 361); fp32 4 million, d = 128, K = 1000 434 398.  Rows of 192 bytes, 4 million 225 220; of 96
// 324 331; of 64 241 250.  A smaller X, fits: 2^20, d = 128, K = 1024 (256 MiB) 1249 1280; fp32 300000, d = 96, K = 400 388 398;
// ragged rows: 12 million, d = 17, K = 600 403 438.
static bool reads_once(const Geometry& g) {
    const int64_t row = (int64_t)g.d * elem_size(g.t);
    return g.len == g.d && row >= 128 && (int64_t)g.B * g.N * row > device_info().llc_bytes;
}

fk_status launch_segment_reduce(const Geometry& g, const Workspace& w, const void* X,
                                const int32_t* sorted_idx, const int32_t* seg_off,
                                const int32_t* item_off, hipStream_t s) {
    const int epl = g.t == FK_F32 ? 4 : 8;
    int lpr_log2 = ceil_log2((int)cdiv(g.d, epl));
    if (lpr_log2 > 6) lpr_log2 = 6;          // wider rows go column block by column block
    const bool wide = g.waves_per_item == 4;
    dim3 grid((unsigned)(wide ? g.max_items : cdiv(g.max_items, 4)), g.B), block(256);
    const bool once = reads_once(g);
#define FK_REDUCE_W(EPL, BF, RAGGED, ONCE) (wide ? segment_reduce_kernel<EPL, BF, 4, RAGGED, ONCE> : segment_reduce_kernel<EPL, BF, 1, RAGGED, ONCE>)
#define FK_REDUCE(EPL, BF)                                                                        \
    do {                                                                                          \
        auto kern = g.len != g.d ? FK_REDUCE_W(EPL, BF, true, false)                              \
                  : once ? FK_REDUCE_W(EPL, BF, false, true) : FK_REDUCE_W(EPL, BF, false, false);  \
        hipLaunchKernelGGL(kern, grid, block, 0, s, X, sorted_idx, seg_off, item_off, w.partial, g.N, g.d, g.K,     \
                           g.rows_per_item, g.max_items, lpr_log2, g.len, item_balance(g));                               \
    } while (0)
    if (g.t == FK_F32) FK_REDUCE(4, false);
    else if (g.t == FK_F16) FK_REDUCE(8, false);
    else FK_REDUCE(8, true);
#undef FK_REDUCE
#undef FK_REDUCE_W
    FK_HIP(hipGetLastError());
    return FK_OK;
}

static EmitTo emit_args(const Geometry& g, const FinalizeArgs& a) {
    EmitTo to;
    to.C_prev = a.C_prev_f32;
    to.C_out = a.C_out_f32;
    to.C_lp_out = g.t == FK_F32 ? nullptr : (uint16_t*)a.C_out_lp;
    to.C_lp_f32_out = g.t != FK_F32 || a.C_out_lp == a.C_out_f32 ? nullptr : (float*)a.C_out_lp;
    to.c_frag = g.t == FK_F32 ? nullptr : (uint16_t*)a.c_frag;
    to.c_bias = a.c_bias;
    to.counts = a.counts;
    to.sums = a.sums;
    to.late_sums = a.late_sums;
    to.late_counts = a.late_counts;
    to.d = g.d; to.K = g.K; to.B = g.B; to.ktiles = g.ktiles; to.dch = g.dchunks;
    to.accumulate = a.accumulate ? 1 : 0;
    to.normalise = a.normalise ? 1 : 0;
    to.bf = g.t == FK_BF16 ? 1 : 0;
    to.late = a.late;
    to.row_len = g.len;
    to.c_split = (uint16_t*)a.c_split;
    to.shift = a.shift;
    to.c2 = a.c2;
    to.list_len = a.list_len;
    to.pair_len = a.pair_len;
    return to;
}

template <int EPL, bool BF, int WAVES>
static fk_status launch_gather_w(const Geometry& g, const Workspace& w, const void* X, const int32_t* assign,
                                 const EmitTo& to, int G, bool merged, hipStream_t s) {
    const int lpr_log2 = std::min(6, ceil_log2((int)cdiv(g.d, EPL)));
    auto kern = g.len == g.d ? gather_update_kernel<EPL, BF, false, WAVES> : gather_update_kernel<EPL, BF, true, WAVES>;
    hipLaunchKernelGGL(kern, dim3((unsigned)((int64_t)g.K * G), g.B), dim3(WAVES * 64), 0, s, X, assign, to, w.partial,
                       w.gather_counts, g.N, G, merged ? 1 : 0, lpr_log2);
    FK_HIP(hipGetLastError());
    return FK_OK;
}

fk_status launch_gather_update(const Geometry& g, const Workspace& w, const void* X, const int32_t* assign,
                               const FinalizeArgs& a, hipStream_t s) {
    const int G = g.gather_parts;
    const bool merged = gather_needs_merge(g, a);
    const EmitTo to = emit_args(g, a);
    // four waves where many workgroups have little to read (32 instances of 1000 points, d = 64, K = 32: 6.6 us, with eight 10.1;
    // 1000, K = 900: 6.2, 9.4)
    const int64_t workgroups = (int64_t)g.B * g.K * G;
    const bool wide = workgroups <= 512 || cdiv(g.N, G) > 1024;
    if (g.t == FK_F32) return (wide ? launch_gather_w<4, false, 8> : launch_gather_w<4, false, 4>)(g, w, X, assign, to, G, merged, s);
    if (g.t == FK_F16) return (wide ? launch_gather_w<8, false, 8> : launch_gather_w<8, false, 4>)(g, w, X, assign, to, G, merged, s);
    return (wide ? launch_gather_w<8, true, 8> : launch_gather_w<8, true, 4>)(g, w, X, assign, to, G, merged, s);
}

// The same for many clusters of few partial rows each (see launch_finalize), in core: a wave per cluster and
// four to a workgroup, sums, centroid and squared norm in registers, so that every read and write is one
// instruction and no barrier lies in the chain of latencies that bounds this.  32 instances, d = 64, K = 8192 132 us -> 92; 32, d = 128, K = 256, eight rows each 14.2 -> 11.6.
// The slots' sums are added one after the other as finalize_kernel's single wave does, so that rows read as stored and padded ones, and
// a fit's last iteration and those that write split centroids, give the same bits.
template <bool RAGGED>
__global__ __launch_bounds__(256) void finalize_wave_kernel(const float* __restrict__ partial, const int32_t* __restrict__ seg_off,
                                                            const int32_t* __restrict__ item_off, EmitTo to, int R, float balance,
                                                            int64_t max_items, const int32_t* __restrict__ wg_counts, int G) {
    const int d = to.d, K = to.K, lane = threadIdx.x & 63;
    const int b = blockIdx.y, k = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
    if (k >= K) return;
    int lr_log2 = 0;
    while ((4 << lr_log2) < d) ++lr_log2;
    const int LR = 1 << lr_log2, slots = 64 >> lr_log2, slot = lane >> lr_log2, col = (lane & (LR - 1)) * 4;
    int i0, i1, n;
    if (wg_counts) {
        i0 = k * G;
        i1 = i0 + G;
        n = 0;
        for (int g = lane; g < G; g += 64) n += wg_counts[((size_t)b * K + k) * G + g];
    } else {
        seg_off += (size_t)b * (K + 1);
        item_off += (size_t)b * (K + 1);
        i0 = item_off[k];
        n = seg_off[k + 1] - seg_off[k];
        const int length = item_length(n, R, balance);
        i1 = length == R ? item_off[k + 1] : i0 + (n + length - 1) / length;
    }
    // eight rows in flight per lane, the eight sums and then the slots' added in a fixed order
    const float* P = partial + (size_t)b * max_items * d;
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    if (col < d) {
        floatx4 a8[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) a8[u] = floatx4{0.f, 0.f, 0.f, 0.f};
        for (int it = i0 + slot; it < i1; it += 8 * slots) {
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int r = it + u * slots;
                if (r < i1) a8[u] += *(const floatx4*)(P + (size_t)r * d + col);
            }
        }
        acc = ((a8[0] + a8[1]) + (a8[2] + a8[3])) + ((a8[4] + a8[5]) + (a8[6] + a8[7]));
    }
    if (wg_counts)
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o);
    floatx4 total;
#pragma unroll
    for (int e = 0; e < 4; ++e) total[e] = __shfl(acc[e], lane & (LR - 1));
    for (int q = 1; q < slots && q < i1 - i0; ++q) {
#pragma unroll
        for (int e = 0; e < 4; ++e) total[e] += __shfl(acc[e], (q << lr_log2) + (lane & (LR - 1)));
    }
    // slots 0 and 1 end two of a lane's four features each; past the end of a caller's row everything is zero
    const bool second = (slot & 1) != 0, mine = slot < 2 && col < d;
    const int j = col + (second ? 2 : 0);
    const int len = RAGGED ? to.row_len : d;
    const size_t at = ((size_t)b * K + k) * len + j;
    const bool here[2] = {mine && (!RAGGED || j < len), mine && (!RAGGED || j + 1 < len)};
    floatx2 c = {0.f, 0.f};
    if (n > 0) {
        c[0] = (float)((double)(second ? total[2] : total[0]) / (double)n);
        c[1] = (float)((double)(second ? total[3] : total[1]) / (double)n);
        if (RAGGED) {
            if (!here[0]) c[0] = 0.f;
            if (!here[1]) c[1] = 0.f;
        }
    } else if (RAGGED) {
        if (here[0]) c[0] = to.C_prev[at];
        if (here[1]) c[1] = to.C_prev[at + 1];
    } else if (mine) {
        c = *(const floatx2*)(to.C_prev + at);
    }
    const uint16_t lp[2] = {float_to_lp(c[0], to.bf), float_to_lp(c[1], to.bf)};
    const uint32_t packed = lp[0] | (uint32_t)lp[1] << 16;
    if (RAGGED) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            if (!here[e]) continue;
            to.C_out[at + e] = c[e];
            if (to.C_lp_out) to.C_lp_out[at + e] = lp[e];
            if (to.C_lp_f32_out) to.C_lp_f32_out[at + e] = c[e];
        }
    } else if (mine) {
        *(floatx2*)(to.C_out + at) = c;
        if (to.C_lp_out) *(uint32_t*)(to.C_lp_out + at) = packed;
        if (to.C_lp_f32_out) *(floatx2*)(to.C_lp_f32_out + at) = c;
    }
    if (lane == 0) to.counts[(size_t)b * K + k] = n;
    if (!to.c_frag) return;
    if (mine)      // fragment order, see emit_centroid
        *(uint32_t*)(to.c_frag + ((((size_t)b * to.ktiles + (k >> 5)) * to.dch + (j >> 4)) * 64 + (((j >> 3) & 1) << 5) + (k & 31)) * 8 +
                     (j & 7)) = packed;
    // the norm as emit_centroid adds it: groups of 8 features one after the other (of an even lane's slots 0 and 1, then of its odd
    // neighbour's), then the groups in order
    float sq[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const float f = lp_to_float(lp[e], to.bf);
        sq[e] = __fmul_rn(f, f);
    }
    float ss = __fadd_rn(sq[0], sq[1]);
#pragma unroll
    for (int q = 0; q < 3; ++q) ss = __fadd_rn(__fadd_rn(__shfl_xor(ss, q == 1 ? LR ^ 1 : LR), sq[0]), sq[1]);
    float n2 = 0.f;
    for (int g0 = 0; g0 * 8 < d; ++g0) n2 = __fadd_rn(n2, __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(ss), LR + 2 * g0 + 1)));
    if (lane == 0) to.c_bias[(size_t)b * to.ktiles * 32 + k] = -0.5f * n2;
}

fk_status launch_finalize(const Geometry& g, const Workspace& w, const int32_t* seg_off,
                          const int32_t* item_off, const FinalizeArgs& a, hipStream_t s,
                          const int32_t* wg_counts, int wg_per_cluster) {
    const int threads = merge_threads(g);
    // A wave per cluster: where merge_threads says so, and where a pass left every cluster up to sixteen rows, one batch of
    // loads, and there are more than four clusters to a compute unit.  us, a workgroup per cluster / so, four iterations: 32 instances of
    // 3000 points, d = 40, K = 100 84 / 70 (the merge 9.2 -> 5.6), 16 of 20000, d = 128, K = 200 218 / 207, 32 of 20000, K = 40 245.4 / 243.6;
    // but 32, K = 16 140.6 / 141.2, 16, d = 64, K = 64 102.3 / 102.9; with 32 rows each 8 of 30000, K = 100 142 / 151.
    // (A one-pass update only: all iterations of a fit take it or none.)
    const bool one_batch = wg_counts && wg_counts == w.wg_counts && g.d <= 128 && wg_per_cluster <= 16 && (int64_t)g.K * g.B > 4 * device_cu_count();
    if ((threads == 64 || one_batch) && a.late == 0 && !a.sums && a.normalise && !a.c_split) {
        auto wave_kernel = g.len == g.d ? finalize_wave_kernel<false> : finalize_wave_kernel<true>;
        hipLaunchKernelGGL(wave_kernel, dim3((unsigned)cdiv(g.K, 4), g.B), dim3(256), 0, s, w.partial, seg_off, item_off,
                           emit_args(g, a), g.rows_per_item, item_balance(g), g.max_items, wg_counts, wg_per_cluster);
        FK_HIP(hipGetLastError());
        return FK_OK;
    }
    const size_t lds = ((size_t)4 * threads + g.d) * sizeof(float);
    // (parts that wait and split centroids never come together: the one is out of core, the other in core)
    const bool ragged = g.len != g.d;
    auto kern = a.late > 0  ? (ragged ? finalize_kernel<true, true, false> : finalize_kernel<true, false, false>)
                : a.c_split ? (ragged ? finalize_kernel<false, true, true> : finalize_kernel<false, false, true>)
                            : (ragged ? finalize_kernel<false, true, false> : finalize_kernel<false, false, false>);
    hipLaunchKernelGGL(kern, dim3(g.K, g.B), dim3(threads), lds, s, w.partial, seg_off, item_off, emit_args(g, a),
                       g.rows_per_item, item_balance(g), g.max_items, wg_counts, wg_per_cluster);
    FK_HIP(hipGetLastError());
    return FK_OK;
}

}  // namespace fk
