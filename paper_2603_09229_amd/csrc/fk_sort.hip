// Inverse mapping of the sort-inverse update (paper Section 4.2, Algorithm 3, first two
// lines): a stable argsort of the assignment vector by cluster id, done as a counting
// sort (one pass when K <= 2048 bins, two least-significant-digit passes above that).
//
// The paper treats argsort as a given primitive.  Here the exclusive scan of the cluster
// histogram doubles as the segment table: seg_off[k] .. seg_off[k+1] is cluster k's run in
// sorted order, so the sorted id sequence is only materialised by the two-pass variant.
// Stability makes point indices ascend inside a segment, which keeps the later row gather
// monotone in address.
//
// Only integer LDS counters are used; no floating-point data is touched here.
#include <stdlib.h>

#include "fk_common.h"

namespace fk {

namespace {

__device__ __forceinline__ int clamp_key(int k, int kmax) { return min(max(k, 0), kmax); }

// For each of a wave's batches of 64 digits, the lanes with the same digit as this one, among the valid
// ones: bit by bit, each bit of all batches before the next, so that a step is one ballot and two three-input
// operations a batch and the batches do not wait for each other (bit by bit inside a batch, with a test of
// the number of bits at each: 6900 of the scatter's 25000 cycles at 300000 keys, K = 400).
template <int kBatches>
__device__ __forceinline__ void match_digits(const int (&digit)[kBatches], int nbits, uint32_t (&lo)[kBatches],
                                             uint32_t (&hi)[kBatches]) {
    for (int b = 0; b < nbits; ++b) {
#pragma unroll
        for (int j = 0; j < kBatches; ++j) {
            const int set = __builtin_amdgcn_sbfe(digit[j], b, 1);       // all ones where the bit is set
            const uint64_t bal = __ballot(set != 0);
            lo[j] &= ~((uint32_t)bal ^ (uint32_t)set);
            hi[j] &= ~((uint32_t)(bal >> 32) ^ (uint32_t)set);
        }
    }
}

__device__ __forceinline__ int lanes_below(uint32_t lo, uint32_t hi) {
    return __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0));
}

// Inclusive scan over the wave in six register moves (row shifts, then the rows' last lanes to those after).
__device__ __forceinline__ int wave_inclusive_scan(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);
    return x;
}

// In-place exclusive scan of v[0..n) in LDS by the whole workgroup; returns the total.
// `scratch` holds at least one int per wave.  Ends with a barrier.
__device__ int block_exclusive_scan(int* v, int n, int* scratch) {
    const int T = blockDim.x, tid = threadIdx.x;
    const int per = (n + T - 1) / T;
    const int lo = min(n, tid * per), hi = min(n, lo + per);
    int sum = 0;
    for (int i = lo; i < hi; ++i) sum += v[i];
    const int inc = wave_inclusive_scan(sum), lane = tid & 63, wave = tid >> 6;
    if (lane == 63) scratch[wave] = inc;
    __syncthreads();
    const int nw = (T + 63) >> 6;
    int before = 0, total = 0;
    for (int w = 0; w < nw; ++w) {
        const int t = scratch[w];
        before += w < wave ? t : 0;
        total += t;
    }
    int run = before + inc - sum;
    for (int i = lo; i < hi; ++i) { const int t = v[i]; v[i] = run; run += t; }
    __syncthreads();
    return total;
}

// The same for the bin totals, by the sort's first workgroup with the tables that follow from them: seg_off[0..n] as the
// scan itself, item_off[0..n] (where not NULL) as the exclusive scan of ceil(v / R).
__device__ void block_scan_tables(int* v, int n, int* scratch, int R, int32_t* seg_off, int32_t* item_off) {
    const int T = blockDim.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int per = (n + T - 1) / T;
    const int lo = min(n, tid * per), hi = min(n, lo + per);
    int sum = 0, items = 0;
    for (int i = lo; i < hi; ++i) {
        sum += v[i];
        items += (v[i] + R - 1) / R;
    }
    const int inc = wave_inclusive_scan(sum), inc_items = wave_inclusive_scan(items);
    if (lane == 63) { scratch[wave] = inc; scratch[16 + wave] = inc_items; }
    __syncthreads();
    int run = inc - sum, run_items = inc_items - items, total = 0, total_items = 0;
    for (int w = 0; w < (T + 63) >> 6; ++w) {
        const int t = scratch[w], ti = scratch[16 + w];
        run += w < wave ? t : 0;
        run_items += w < wave ? ti : 0;
        total += t;
        total_items += ti;
    }
    for (int i = lo; i < hi; ++i) {
        const int t = v[i];
        v[i] = run;
        seg_off[i] = run;
        if (item_off) item_off[i] = run_items;
        run += t;
        run_items += (t + R - 1) / R;
    }
    if (tid == 0) {
        seg_off[n] = total;
        if (item_off) item_off[n] = total_items;
    }
    __syncthreads();
}

}  // namespace

// ------------------------------------------------------------------------------------
// Tiling shared by the histogram and scatter kernels: a workgroup of WAVES waves (8, or 4
// when the per-wave counters of a wide digit would not fit in LDS) owns `rounds` consecutive
// sub-tiles of 4096 keys.  With one round, wave w owns 4096/WAVES consecutive keys as batches
// of 64, batch j at offset j*64 + lane; with several, the scatter gives each wave `rounds` such
// runs back to back (the histogram only counts, any partition of the tile serves it).  All
// loads of a round are issued before any is used.
constexpr int kSubTile = 4096;

// Keys come back clamped to [0, kmax]; -1 marks a lane past the end of the array.
template <int kBatches, typename Key>
__device__ __forceinline__ void load_round(const Key* __restrict__ keys, int64_t base,
                                           int64_t N, int lane, int kmax, int (&k)[kBatches]) {
#pragma unroll
    for (int j = 0; j < kBatches; ++j) {
        const int64_t i = base + j * 64 + lane;
        k[j] = i < N ? keys[i] : -1;
    }
#pragma unroll
    for (int j = 0; j < kBatches; ++j) {
        const int64_t i = base + j * 64 + lane;
        k[j] = i < N ? clamp_key(k[j], kmax) : -1;
    }
}

// Per-workgroup digit histogram, written transposed, H[b][bin][blk], for the scan kernel, or
// (by_block) H[b][blk][bin] for scatter workgroups that add the earlier ones' up themselves.
template <int kSortWaves, typename Key>
__global__ __launch_bounds__(kSortWaves * 64) void sort_hist_kernel(
    const Key* __restrict__ keys, int32_t* __restrict__ H, int64_t N, int rounds, int NB,
    int shift, int mask, int kmax, int nbits, int by_block) {
    constexpr int kSortThreads = kSortWaves * 64, kBatches = kSubTile / kSortThreads;
    extern __shared__ int lds[];
    int* hist = lds;
    const int b = blockIdx.y, blk = blockIdx.x, nb = gridDim.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    keys += (size_t)b * N;
    // Few bins: hot bins would serialise the LDS adds of a wave (lanes hitting one address are
    // processed one after the other), so each group of lanes (lane % 16) counts into its own
    // copy of the histogram and the copies are added at the end.
    const int copies = NB <= 64 ? 16 : 1;
    int* my_hist = hist + (copies > 1 ? (lane & 15) * NB : 0);
    for (int i = tid; i < NB * copies; i += kSortThreads) hist[i] = 0;
    __syncthreads();
    // rounds are software-pipelined: the next round's keys are requested before this round's
    // are counted
    const int64_t base0 = (int64_t)blk * rounds * kSubTile + wave * (kBatches * 64);
    int k[kBatches], kn[kBatches];
    load_round(keys, base0, N, lane, kmax, k);
    for (int r = 0; r < rounds; ++r) {
        const int64_t nbase = base0 + (int64_t)(r + 1) * kSubTile;
        const bool more = r + 1 < rounds && nbase < N;
        if (more) load_round(keys, nbase, N, lane, kmax, kn);
        // one LDS add per key (cheaper than resolving duplicates with ballots first)
#pragma unroll
        for (int j = 0; j < kBatches; ++j)
            if (k[j] >= 0) atomicAdd(&my_hist[(k[j] >> shift) & mask], 1);
        if (!more) break;
#pragma unroll
        for (int j = 0; j < kBatches; ++j) k[j] = kn[j];
    }
    __syncthreads();
    int32_t* out = H + (size_t)b * NB * nb + (by_block ? (size_t)blk * NB : (size_t)blk);
    const size_t step = by_block ? 1 : nb;
    for (int i = tid; i < NB; i += kSortThreads) {
        int c = 0;
        for (int q = 0; q < copies; ++q) c += hist[q * NB + i];
        out[(size_t)i * step] = c;
    }
}

// Exclusive scan of H[b][bin][0..nb) in place; tot[b][bin] = row sum.  TPB threads (one wave,
// or the whole workgroup for long rows) share a bin, each owning a contiguous run of entries.
template <int TPB>
__global__ __launch_bounds__(256) void sort_binscan_kernel(int32_t* __restrict__ H,
                                                           int32_t* __restrict__ tot, int nb,
                                                           int NB) {
    __shared__ int wsum[4];
    const int b = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int bin = TPB == 64 ? blockIdx.x * 4 + wave : blockIdx.x;
    const int t = TPB == 64 ? lane : threadIdx.x;          // index inside the bin's team
    const bool live = bin < NB;
    int32_t* row = H + ((size_t)b * NB + (live ? bin : 0)) * nb;
    const int per = (nb + TPB - 1) / TPB;
    const int lo = live ? min(nb, t * per) : 0, hi = live ? min(nb, lo + per) : 0;
    int sum = 0;
    for (int i = lo; i < hi; ++i) sum += row[i];
    const int inc = wave_inclusive_scan(sum);
    int base = 0, total = inc;                             // total valid in lane 63
    if (TPB == 256) {
        if (lane == 63) wsum[wave] = inc;
        __syncthreads();
        for (int w = 0; w < wave; ++w) base += wsum[w];
        total = wsum[0] + wsum[1] + wsum[2] + wsum[3];
        if (live && threadIdx.x == 0) tot[(size_t)b * NB + bin] = total;
    } else if (live && lane == 63) {
        tot[(size_t)b * NB + bin] = total;
    }
    int run = base + inc - sum;
    for (int i = lo; i < hi; ++i) {
        const int v = row[i];
        row[i] = run;
        run += v;
    }
}

// Stable scatter.  Waves walk their keys in input order, so equal keys keep their order.
//   vals_in == NULL: values are the key positions (first pass).
//   kScans: see sort_scatter_scans; rounds is 1.  An instantiation of its own: the code costs the others 2%
//   when it is only skipped.  Both of eight waves are held to 80 registers, of which they spill 4 and 2 (three workgroups on
//   a compute unit; fk_sort_inverse, us, held / not: 2^23 keys, K = 4096 110 / 121, 2^22, K = 32 25.7 / 27.4, 2^25, K = 300 302 / 306;
//   300000, K = 400 15.8 / 15.2, 70001, K = 333 13.3 / 12.9, where there are few workgroups).  That of four is not: held to three
//   waves per SIMD 2^20 keys, K = 2000 took 39.4 instead of 39.1, 100000 23.3 instead of 22.7.
// Bound by its chain of latencies: keys and tables, ranks, two scans, LDS, stores.  300000 keys, K = 400 11.7 -> 9.1
// us, 2^20, K = 1024 15.5 -> 13.0, 2^23 in two passes of 64 bins 84.7 -> 73.6, all together, since the tables are requested with the
// keys, the ranks found bit by bit for all batches at once (2.9 us of the first), the scans in register moves, both
// tables of the first workgroup in one scan, and each loop over LDS reads before it writes.
//   keys_out may be NULL.  seg_off / item_off are written by workgroup 0 when non-NULL
//   (single-pass sort: bins are cluster ids, so the bin offsets are the segment table).
//   Key: the ids as the caller has them, or the 16-bit copies (K is at most 65536) that a first pass leaves for the second:
//   2^23 keys, K = 4096, both histograms, both scatters, boundaries 27 + 73 + 11 us -> 20 + 61 + 6; evenly drawn ids, fk_sort_inverse there
//   110 -> 95, fk_update, d = 128, 494 -> 480, 2^25 x 16 1139 -> 1028, 30000 x 64, K = 5000 44 -> 42.
template <int kSortWaves, bool kScans, typename Key>
__global__ __launch_bounds__(kSortWaves * 64, kSortWaves == 8 ? 6 : 1) void sort_scatter_kernel(
    const Key* __restrict__ keys, const int32_t* __restrict__ vals_in,
    const int32_t* __restrict__ H, const int32_t* __restrict__ tot,
    int32_t* __restrict__ vals_out, uint16_t* __restrict__ keys_out,
    int32_t* __restrict__ seg_off, int32_t* __restrict__ item_off, int64_t N, int rounds,
    int NB, int shift, int mask, int kmax, int nbits, int R, int staged, int solo) {
    constexpr int kSortThreads = kSortWaves * 64, kBatches = kSubTile / kSortThreads;
    extern __shared__ int lds[];
    int* off = lds;                    // [NB]
    int* scratch = off + NB;           // [40]
    int* wcnt = scratch + 40;          // [kSortWaves][NB]
    // staged only: [NB] bin starts, then the tile's keys and values in sorted order
    int* gdel = wcnt + kSortWaves * NB;
    int* skey = gdel + NB;
    int* sval = skey + kSubTile;
    const int b = blockIdx.y, blk = blockIdx.x, nb = gridDim.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    keys += (size_t)b * N;
    if (vals_in) vals_in += (size_t)b * N;
    vals_out += (size_t)b * N;
    if (keys_out) keys_out += (size_t)b * N;
    tot += (size_t)b * NB;
    H += (size_t)b * NB * nb + (kScans ? 0 : blk);

    // The first round's keys and the tables are requested before anything waits for them.  A wave owns
    // `rounds` consecutive batches-of-8 (contiguous in the input, so that wave order
    // is input order and the sort stays stable with several rounds)
    int k[kBatches];
    const int64_t base0 = (int64_t)blk * rounds * kSubTile + (int64_t)wave * rounds * (kBatches * 64);
    constexpr int kRoundStep = kBatches * 64;
#pragma unroll
    for (int j = 0; j < kBatches; ++j) {
        const int64_t i = base0 + j * 64 + lane;
        k[j] = i < N ? keys[i] : 0;
    }
    // this workgroup's column of the scanned histogram table (one entry per bin, a cache line
    // apart), needed only after the counting pass, and the bin totals
    constexpr int kHPer = (kSortWaves == 8 ? 1024 : 2048) / kSortThreads;      // (eight waves: at most 1024 bins)
    int hcol[kHPer], bin_total[kHPer];
    if constexpr (kScans) {
        // Few sort workgroups: no scan kernel has run; each workgroup adds up the counts of the earlier
        // ones (where its own keys start inside the bins) and of all of them (the bin totals) for itself.
#pragma unroll
        for (int q = 0; q < kHPer; ++q) {
            const int i = tid + q * kSortThreads;
            int before = 0, all = 0;
            if (i < NB) {
#pragma unroll 8
                for (int o = 0; o < nb; ++o) {
                    const int c = H[(size_t)o * NB + i];
                    all += c;
                    before += o < blk ? c : 0;
                }
            }
            hcol[q] = before;
            bin_total[q] = all;
        }
    } else {
#pragma unroll
        for (int q = 0; q < kHPer; ++q) {
            const int i = tid + q * kSortThreads;
            const bool live = !solo && i < NB;
            hcol[q] = live ? H[(size_t)i * nb] : 0;
            bin_total[q] = live ? tot[i] : 0;
        }
    }
    for (int i = tid; i < kSortWaves * NB; i += kSortThreads) wcnt[i] = 0;

    // Bin totals -> off[] (exclusive scan: where each bin starts in the output), plus the
    // segment and item tables when asked for.  The totals come from the scan kernel, or, when
    // one workgroup sorts the whole instance (solo), from its own per-wave counts after the
    // counting pass -- no histogram or scan kernel runs then.
    auto offsets_from_totals = [&]() {
#pragma unroll
        for (int q = 0; q < kHPer; ++q) {
            const int i = tid + q * kSortThreads;
            if (i < NB) {
                int t = bin_total[q];
                if (!kScans && solo) {
#pragma unroll
                    for (int w = 0; w < kSortWaves; ++w) t += wcnt[w * NB + i];
                }
                off[i] = t;
            }
        }
        __syncthreads();
        if (seg_off && blk == 0)
            block_scan_tables(off, NB, scratch, R, seg_off + (size_t)b * (NB + 1), item_off ? item_off + (size_t)b * (NB + 1) : nullptr);
        else
            (void)block_exclusive_scan(off, NB, scratch);
    };
    if (kScans || !solo) offsets_from_totals();
    else __syncthreads();
#pragma unroll
    for (int j = 0; j < kBatches; ++j) {
        const int64_t i = base0 + j * 64 + lane;
        k[j] = i < N ? clamp_key(k[j], kmax) : -1;
    }

    int* mine = wcnt + wave * NB;
    // info[j] = rank among equal digits of the batch | (size of that group << 8)
    int info[kBatches];

    if (kScans || rounds == 1) {
        // Keys, ranks and each key's position inside its wave's run of the digit stay in
        // registers between the two passes.  Pass 1: every lane reads the wave's running count
        // of its digit, then the first lane of each group of equal digits adds the group's
        // size; LDS executes a wave's operations in order, so the eight batches need no wait
        // between them.
        int pre[kBatches], digit[kBatches];
        uint32_t lo[kBatches], hi[kBatches];
#pragma unroll
        for (int j = 0; j < kBatches; ++j) {
            const uint64_t valid = __ballot(k[j] >= 0);
            digit[j] = k[j] >= 0 ? (k[j] >> shift) & mask : 0;
            lo[j] = (uint32_t)valid;
            hi[j] = (uint32_t)(valid >> 32);
        }
        match_digits(digit, nbits, lo, hi);
#pragma unroll
        for (int j = 0; j < kBatches; ++j) {
            info[j] = lanes_below(lo[j], hi[j]);
            pre[j] = k[j] >= 0 ? mine[digit[j]] : 0;
            __builtin_amdgcn_wave_barrier();
            if (k[j] >= 0 && info[j] == 0) atomicAdd(&mine[digit[j]], __popc(lo[j]) + __popc(hi[j]));
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        if (!kScans && solo) offsets_from_totals();
        int v[kBatches];
        if (vals_in) {
#pragma unroll
            for (int j = 0; j < kBatches; ++j) {
                const int64_t i = base0 + j * 64 + lane;
                v[j] = i < N ? vals_in[i] : 0;
            }
        }
        if (staged) {
            // Few bins, long runs: the tile is first put in sorted order in LDS and then
            // written by consecutive threads, so that a store instruction covers a few
            // contiguous runs instead of 64 scattered words.
            for (int i = tid; i < NB; i += kSortThreads) {
                int run = 0, t[kSortWaves];
#pragma unroll
                for (int w = 0; w < kSortWaves; ++w) t[w] = wcnt[w * NB + i];
#pragma unroll
                for (int w = 0; w < kSortWaves; ++w) {
                    wcnt[w * NB + i] = run;           // where wave w's run starts inside the bin's
                    run += t[w];
                }
                gdel[i] = run;                        // the tile's count of bin i
            }
            __syncthreads();
            block_exclusive_scan(gdel, NB, scratch);  // -> where bin i starts inside the tile
#pragma unroll
            for (int j = 0; j < kBatches; ++j) {
                if (k[j] >= 0) {
                    const int digit = (k[j] >> shift) & mask;
                    const int lp = gdel[digit] + mine[digit] + pre[j] + info[j];
                    skey[lp] = k[j];
                    sval[lp] = vals_in ? v[j] : (int32_t)(base0 + j * 64 + lane);
                }
            }
            __syncthreads();
            // global position = position in the tile + (global start of the tile's run of the bin
            // - its start inside the tile)
#pragma unroll
            for (int q = 0; q < kHPer; ++q) {
                const int i = tid + q * kSortThreads;
                if (i < NB) gdel[i] = off[i] + hcol[q] - gdel[i];
            }
            __syncthreads();
            const int64_t tile0 = (int64_t)blk * kSubTile;
            const int live = (int)min((int64_t)kSubTile, N - tile0);
            int pos[kBatches];
#pragma unroll
            for (int j = 0; j < kBatches; ++j) {
                const int i = tid + j * kSortThreads;
                k[j] = i < live ? skey[i] : 0;
                info[j] = i < live ? sval[i] : 0;
            }
#pragma unroll
            for (int j = 0; j < kBatches; ++j) pos[j] = tid + j * kSortThreads + gdel[(k[j] >> shift) & mask];
#pragma unroll
            for (int j = 0; j < kBatches; ++j) {
                if (tid + j * kSortThreads < live) {
                    vals_out[pos[j]] = info[j];
                    if (keys_out) keys_out[pos[j]] = (uint16_t)k[j];
                }
            }
            return;
        }
        // counts -> start positions: global bin offset + earlier workgroups + earlier waves
#pragma unroll
        for (int q = 0; q < kHPer; ++q) {
            const int i = tid + q * kSortThreads;
            if (i < NB) {
                int run = off[i] + hcol[q], t[kSortWaves];
#pragma unroll
                for (int w = 0; w < kSortWaves; ++w) t[w] = wcnt[w * NB + i];
#pragma unroll
                for (int w = 0; w < kSortWaves; ++w) {
                    wcnt[w * NB + i] = run;
                    run += t[w];
                }
            }
        }
        __syncthreads();
        // pass 2: position = start of the wave's run + position inside the run
        int start[kBatches];
#pragma unroll
        for (int j = 0; j < kBatches; ++j) start[j] = k[j] >= 0 ? mine[(k[j] >> shift) & mask] : 0;
#pragma unroll
        for (int j = 0; j < kBatches; ++j) {
            if (k[j] >= 0) {
                const int pos = start[j] + pre[j] + info[j];
                vals_out[pos] = vals_in ? v[j] : (int32_t)(base0 + j * 64 + lane);
                if (keys_out) keys_out[pos] = (uint16_t)k[j];
            }
        }
        return;
    }

    // More than one round per workgroup (beyond 16M keys per instance): ranks are recomputed
    // in the second pass and the wave's cursors advance batch by batch.
    auto rank_round = [&](bool count) {
        int digit[kBatches];
        uint32_t lo[kBatches], hi[kBatches];
#pragma unroll
        for (int j = 0; j < kBatches; ++j) {
            const uint64_t valid = __ballot(k[j] >= 0);
            digit[j] = k[j] >= 0 ? (k[j] >> shift) & mask : 0;
            lo[j] = (uint32_t)valid;
            hi[j] = (uint32_t)(valid >> 32);
        }
        match_digits(digit, nbits, lo, hi);
#pragma unroll
        for (int j = 0; j < kBatches; ++j) {
            const int rank = lanes_below(lo[j], hi[j]), cnt = __popc(lo[j]) + __popc(hi[j]);
            info[j] = rank | (cnt << 8);
            if (count && k[j] >= 0 && rank == 0) mine[digit[j]] += cnt;
            __builtin_amdgcn_wave_barrier();
        }
    };
    // pass 1: per-wave digit counts
    rank_round(true);
    for (int r = 1; r < rounds; ++r) {
        const int64_t base = base0 + (int64_t)r * kRoundStep;
        if (base >= N) break;
        load_round(keys, base, N, lane, kmax, k);
        rank_round(true);
    }
    __syncthreads();
    if (!kScans && solo) offsets_from_totals();
    // counts -> start positions: global bin offset + earlier workgroups + earlier waves
#pragma unroll
    for (int q = 0; q < kHPer; ++q) {
        const int i = tid + q * kSortThreads;
        if (i < NB) {
            int run = off[i] + hcol[q];
            for (int w = 0; w < kSortWaves; ++w) {
                const int t = wcnt[w * NB + i];
                wcnt[w * NB + i] = run;
                run += t;
            }
        }
    }
    __syncthreads();
    // pass 2: write, advancing the wave's cursors batch by batch
    for (int r = 0; r < rounds; ++r) {
        const int64_t base = base0 + (int64_t)r * kRoundStep;
        if (base >= N) break;
        load_round(keys, base, N, lane, kmax, k);
        rank_round(false);
        int v[kBatches];
        if (vals_in) {
#pragma unroll
            for (int j = 0; j < kBatches; ++j) {
                const int64_t i = base + j * 64 + lane;
                v[j] = i < N ? vals_in[i] : 0;
            }
        }
#pragma unroll
        for (int j = 0; j < kBatches; ++j) {
            const bool valid = k[j] >= 0;
            const int key = valid ? k[j] : 0;
            const int digit = (key >> shift) & mask;
            const int rank = info[j] & 255, cnt = info[j] >> 8;
            int pos = 0;
            if (valid) pos = mine[digit] + rank;
            __builtin_amdgcn_wave_barrier();
            if (valid) {
                vals_out[pos] = vals_in ? v[j] : (int32_t)(base + j * 64 + lane);
                if (keys_out) keys_out[pos] = (uint16_t)key;
                if (rank == 0) mine[digit] += cnt;
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
}

// Two-pass sort only: segment table from the sorted id sequence.  Position j opens the
// segments of every id in (ks[j-1], ks[j]]; ids above the last key get N.
constexpr int kBoundaryKeys = 1024;      // of a workgroup: four of each thread, requested together
__global__ __launch_bounds__(256) void sort_boundaries_kernel(const uint16_t* __restrict__ ks,
                                                              int32_t* __restrict__ seg_off, int64_t N, int K) {
    const int b = blockIdx.y;
    ks += (size_t)b * N;
    seg_off += (size_t)b * (K + 1);
    const int64_t j0 = (int64_t)blockIdx.x * kBoundaryKeys + threadIdx.x;
    int cur[kBoundaryKeys / 256], prev[kBoundaryKeys / 256];
#pragma unroll
    for (int u = 0; u < kBoundaryKeys / 256; ++u) {
        const int64_t j = j0 + u * 256;
        cur[u] = j < N ? ks[j] : 0;
        prev[u] = j < N && j > 0 ? ks[j - 1] : -1;
    }
#pragma unroll
    for (int u = 0; u < kBoundaryKeys / 256; ++u) {
        const int64_t j = j0 + u * 256;
        if (j >= N) break;
        for (int k = prev[u] + 1; k <= cur[u]; ++k) seg_off[k] = (int32_t)j;
        if (j == N - 1)
            for (int k = cur[u] + 1; k <= K; ++k) seg_off[k] = (int32_t)N;
    }
}

// Two-pass sort only: item_off = exclusive scan of ceil(n_k / R).  Every workgroup of 1024 clusters adds up all those
// before its own, 64 loads of a thread at the most (K = 65536), many in flight and neighbours to neighbours.  (One workgroup whose
// threads each walked K / 1024 neighbours: 113 us at K = 60000, half of an update of 200000 points.)
__global__ __launch_bounds__(1024) void item_offsets_kernel(const int32_t* __restrict__ seg_off,
                                                            int32_t* __restrict__ item_off, int K, int R) {
    __shared__ int before[16], own[16];
    const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    seg_off += (size_t)b * (K + 1);
    item_off += (size_t)b * (K + 1);
    auto items = [&](int k) { return (seg_off[k + 1] - seg_off[k] + R - 1) / R; };
    const int k0 = blockIdx.x * 1024, k = k0 + tid;
    const int mine = k < K ? items(k) : 0;
    int sum = 0;
#pragma unroll 8
    for (int q = tid; q < k0; q += 1024) sum += items(q);
    const int inc = wave_inclusive_scan(mine), earlier = wave_inclusive_scan(sum);
    if (lane == 63) { before[wave] = earlier; own[wave] = inc; }
    __syncthreads();
    int run = inc - mine;
#pragma unroll
    for (int w = 0; w < 16; ++w) run += before[w] + (w < wave ? own[w] : 0);
    if (k < K) item_off[k] = run;
    if (k == K - 1) item_off[K] = run + mine;
}

// ------------------------------------------------------------------------------------
static int ceil_log2(int v) {
    int b = 0;
    while ((1 << b) < v) ++b;
    return b;
}

// upper limit of the LDS-staged scatter, in bins (fk_set_option("sort_stage_bins"); 0 = never)
static std::atomic<int> g_stage_max_bins{1024};

void set_sort_stage_bins(int v) { g_stage_max_bins.store(v < 0 ? 1024 : v, std::memory_order_relaxed); }

template <typename Key>
static fk_status sort_pass(const Geometry& g, const Workspace& w, const Key* keys,
                           const int32_t* vals_in, int32_t* vals_out, uint16_t* keys_out,
                           int32_t* seg_off, int32_t* item_off, int NB, int shift, int mask,
                           hipStream_t s) {
    const int nbits = ceil_log2(NB) < 1 ? 1 : ceil_log2(NB);
    const int rounds = g.sort_tile / kSubTile;
    int32_t* H = w.block_hist;
    int32_t* tot = w.digit_off;
    dim3 grid(g.sort_blocks, g.B);
    // 8 waves of counters would not fit in LDS (ids as they come only: a second pass has at most 256 bins)
    constexpr int kWide = sizeof(Key) == 4 ? 4 : 8;
    const bool wide = kWide == 4 && NB > 1024;
    // one workgroup per instance: the scatter kernel counts for itself
    const int solo = g.sort_blocks == 1 ? 1 : 0;
    const int by_block = rounds == 1 && sort_scatter_scans(g.B, g.sort_blocks, NB) ? 1 : 0;
    if (!solo) {
        const size_t hist_lds = (size_t)NB * (NB <= 64 ? 16 : 1) * sizeof(int);
        if (wide)
            hipLaunchKernelGGL((sort_hist_kernel<kWide, Key>), grid, dim3(256), hist_lds, s, keys, H, g.N,
                               rounds, NB, shift, mask, g.K - 1, nbits, by_block);
        else
            hipLaunchKernelGGL((sort_hist_kernel<8, Key>), grid, dim3(512), hist_lds, s, keys, H, g.N,
                               rounds, NB, shift, mask, g.K - 1, nbits, by_block);
        FK_HIP(hipGetLastError());
        if (!by_block && g.sort_blocks > 512)
            hipLaunchKernelGGL(sort_binscan_kernel<256>, dim3((unsigned)NB, g.B), dim3(256), 0, s, H,
                               tot, g.sort_blocks, NB);
        else if (!by_block)
            hipLaunchKernelGGL(sort_binscan_kernel<64>, dim3((unsigned)cdiv(NB, 4), g.B), dim3(256), 0,
                               s, H, tot, g.sort_blocks, NB);
        FK_HIP(hipGetLastError());
    }
    const int waves = wide ? 4 : 8;
    // One tile per workgroup: sorted in LDS first, then written in contiguous runs.  Measured
    // (2^20 .. 2^25 keys): pays from 32 bins (below that a wave's stores already fall into few
    // runs) up to 1024 (beyond, the LDS footprint costs more than the runs, 1-2 keys, give);
    // 2x on the 64..256-bin passes of the two-pass sort.
    const int staged = rounds == 1 && NB >= 32 && NB <= g_stage_max_bins.load(std::memory_order_relaxed) ? 1 : 0;
    const size_t lds = (size_t)(NB + 40 + waves * NB + (staged ? NB + 2 * kSubTile : 0)) * sizeof(int);
    auto kern = wide ? sort_scatter_kernel<kWide, false, Key> : by_block ? sort_scatter_kernel<8, true, Key> : sort_scatter_kernel<8, false, Key>;
    if (lds > 64 * 1024) {
        static PerDeviceInt attr_set[3];
        PerDeviceInt& set = attr_set[wide ? 0 : 1 + by_block];
        if (!set.get()) {
            FK_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024));
            set.set(1);
        }
    }
    hipLaunchKernelGGL(kern, grid, dim3(waves * 64), lds, s, keys, vals_in, H, tot, vals_out, keys_out, seg_off, item_off,
                       g.N, rounds, NB, shift, mask, g.K - 1, nbits, g.rows_per_item, staged, solo);
    FK_HIP(hipGetLastError());
    return FK_OK;
}

fk_status launch_sort_inverse(const Geometry& g, const Workspace& w, const int32_t* assign,
                              int32_t* sorted_idx, int32_t* seg_off, int32_t* item_off,
                              hipStream_t s) {
    if (g.sort_passes == 1)
        return sort_pass(g, w, assign, nullptr, sorted_idx, nullptr, seg_off, item_off, g.K, 0,
                         0x7FFFFFFF, s);
    const int lb = g.pass_bits[0], hb = g.pass_bits[1];
    fk_status st = sort_pass(g, w, assign, nullptr, w.vals_tmp, w.keys_tmp, nullptr, nullptr,
                             1 << lb, 0, (1 << lb) - 1, s);
    if (st != FK_OK) return st;
    st = sort_pass(g, w, w.keys_tmp, w.vals_tmp, sorted_idx, w.keys_sorted, nullptr, nullptr,
                   1 << hb, lb, (1 << hb) - 1, s);
    if (st != FK_OK) return st;
    hipLaunchKernelGGL(sort_boundaries_kernel, dim3((unsigned)cdiv(g.N, kBoundaryKeys), g.B), dim3(256), 0,
                       s, w.keys_sorted, seg_off, g.N, g.K);
    FK_HIP(hipGetLastError());
    if (item_off) {
        hipLaunchKernelGGL(item_offsets_kernel, dim3((unsigned)cdiv(g.K, 1024), g.B), dim3(1024), 0, s, seg_off, item_off,
                           g.K, g.rows_per_item);
        FK_HIP(hipGetLastError());
    }
    return FK_OK;
}

}  // namespace fk
