// Out-of-core Lloyd iterations: chunked stream overlap (paper Section 4.3).
//
// X stays in pinned host memory.  Two device chunk buffers are filled alternately by
// hipMemcpyAsync on a side stream while the compute stream runs assignment, sort-inverse
// and segment reduction on the other buffer.  Events order the two streams:
//   ready[i]  copy into buffer i finished      (compute waits)
//   freed[i]  compute on buffer i finished     (the next copy into i waits)
// (Small calls copy on the compute stream instead, see below.)
// An iteration after the first starts with the two chunks that are still in the buffers, which saves
// two copies per iteration (all of them with at most two chunks).  The call is bound by its copies
// below about K = 3000 (57 GB/s from the host: 8 chunks of 2^18 x 128 fp16, K = 1024, two
// iterations: 19.5 ms with 16 copies, 17.3 with 14).
// The centroids are frozen for the whole iteration; per-chunk sums and counts are added
// onto running totals and normalised once after the last chunk, so the result is the
// in-core one up to fp32 summation order.  They are added in the order of the chunks whatever the
// order in which the chunks are taken -- those of the chunks taken early wait in two arrays of their
// own until their turn -- so that a call of n iterations gives the bits of n calls of one.
#include "fk_common.h"
#include "fk_device.h"

namespace fk {

// Pinned host memory, read over the host link: every thread asks for up to four pieces at once.
template <typename Piece>
__global__ __launch_bounds__(256) void copy_bytes_kernel(const Piece* __restrict__ src, Piece* __restrict__ dst, uint32_t n) {
    const uint32_t step = gridDim.x * 256;
    for (uint32_t i0 = blockIdx.x * 256 + threadIdx.x; i0 < n; i0 += 4 * step) {
        Piece v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (i0 + u * step < n) v[u] = src[i0 + u * step];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (i0 + u * step < n) dst[i0 + u * step] = v[u];
    }
}

static fk_status launch_copy_bytes(const void* src, void* dst, size_t bytes, hipStream_t s) {
    const size_t aligned = ((uintptr_t)src | bytes) & 15;    // dst is a chunk buffer, and rows are whole elements
    const size_t piece = aligned == 0 ? 16 : (aligned & 3) == 0 ? 4 : 2;
    const uint32_t n = (uint32_t)(bytes / piece);
    const dim3 grid((unsigned)std::min<uint32_t>((n + 255) / 256, 1024));
    if (piece == 16) hipLaunchKernelGGL(copy_bytes_kernel<uintx4>, grid, dim3(256), 0, s, (const uintx4*)src, (uintx4*)dst, n);
    else if (piece == 4) hipLaunchKernelGGL(copy_bytes_kernel<uint32_t>, grid, dim3(256), 0, s, (const uint32_t*)src, (uint32_t*)dst, n);
    else hipLaunchKernelGGL(copy_bytes_kernel<uint16_t>, grid, dim3(256), 0, s, (const uint16_t*)src, (uint16_t*)dst, n);
    FK_HIP(hipGetLastError());
    return FK_OK;
}

struct OocLayout {
    size_t chunk_bytes;   // one chunk buffer
    size_t core_bytes;    // in-core workspace for one chunk
    size_t assign_bytes;  // per-chunk assignment buffer (used when the caller keeps none)
    size_t total;         // what the call cannot do without
    size_t late_sum_bytes, late_count_bytes;   // sums and counts of a chunk taken early
    size_t with_late;     // ... with room for two of them: the size that is asked for.  In less room the
                          // chunks are taken in order and copied in every iteration
};

static bool ooc_layout(int64_t chunk_rows, int d, int K, fk_dtype t, OocLayout* L, Geometry* g) {
    if (!make_geometry(1, chunk_rows, d, K, t, g)) return false;
    (void)limit_gather_parts(g);              // the chunks that fit a given dev_ws are those that sorting has room for
    // chunk buffers have room for rows of the kernels' width (a multiple of 8), which rows of fewer
    // than 8 elements need: they land in them through a pitched copy, the padding columns zeroed once
    L->chunk_bytes = align_up((size_t)chunk_rows * g->d * elem_size(t), 256);
    L->core_bytes = align_up(carve(*g, nullptr, false).bytes, 256);
    L->assign_bytes = align_up((size_t)chunk_rows * 4, 256);
    L->total = 2 * L->chunk_bytes + L->core_bytes + L->assign_bytes;
    L->late_sum_bytes = (size_t)K * g->d * 4;
    L->late_count_bytes = (size_t)K * 4;
    L->with_late = L->total + align_up(2 * L->late_sum_bytes, 256) + align_up(2 * L->late_count_bytes, 256);
    return true;
}

}  // namespace fk

using namespace fk;

extern "C" {

size_t fk_ooc_workspace_bytes(int64_t chunk_rows, int d, int K, fk_dtype t) {
    OocLayout L;
    Geometry g;
    if (chunk_rows < 1 || !ooc_layout(chunk_rows, d, K, t, &L, &g)) return 0;
    return L.with_late;
}

fk_status fk_lloyd_ooc(const void* X_host, float* C_f32, int32_t* assign, int32_t* counts,
                       int64_t N, int d, int K, fk_dtype t, int iters, int64_t chunk_rows,
                       void* dev_ws, size_t dev_ws_bytes, void* stream) {
    if (N < 1 || d < 1 || K < 1 || iters < 0 || chunk_rows < 0) {
        set_error("fk_lloyd_ooc: N, d, K must be positive, iters and chunk_rows non-negative");
        return FK_EINVAL;
    }
    if (!X_host || !C_f32 || !counts || !dev_ws || ((uintptr_t)dev_ws & 255u) ||
        ((uintptr_t)C_f32 & 15u) || ((uintptr_t)counts & 15u) || ((uintptr_t)assign & 15u) ||
        ((uintptr_t)X_host & 15u)) {
        set_error("fk_lloyd_ooc: NULL or misaligned pointer");
        return FK_EINVAL;
    }
    bool pinned_here = false;                    // through the current device
    {
        // X_host must be pinned (page-locked) host memory: from pageable memory hipMemcpyAsync
        // stages through a bounce buffer and the copies no longer overlap the kernels.  Both ends
        // of the array are looked up.
        const size_t bytes = (size_t)N * (size_t)d * elem_size(t);
        const char* ends[2] = {(const char*)X_host, (const char*)X_host + (bytes ? bytes - 1 : 0)};
        pinned_here = true;
        for (const char* p : ends) {
            hipPointerAttribute_t attr;
            const hipError_t pe = hipPointerGetAttributes(&attr, p);
            if (pe != hipSuccess) {
                (void)hipGetLastError();      // an unknown pointer is reported as an error: clear it
                set_error("fk_lloyd_ooc: X_host is not pinned host memory (the HIP runtime does not know the pointer: %s)",
                          hipGetErrorString(pe));
                return FK_EINVAL;
            }
            if (attr.type != hipMemoryTypeHost) {
                set_error("fk_lloyd_ooc: X_host must be pinned host memory (hipHostMalloc), got memory type %d",
                          (int)attr.type);
                return FK_EINVAL;
            }
            pinned_here &= attr.device == current_device();
        }
    }
    Geometry gfull;
    OocLayout L;
    if (chunk_rows == 0) {
        // largest multiple of 1024 rows (or all of N) whose footprint fits
        const int64_t unit = 1024;
        auto largest = [&](bool late) {
            int64_t lo = 0, hi = cdiv(N, unit);
            while (lo < hi) {
                const int64_t mid = (lo + hi + 1) / 2;
                const int64_t rows = mid * unit < N ? mid * unit : N;
                if (ooc_layout(rows, d, K, t, &L, &gfull) && (late ? L.with_late : L.total) <= dev_ws_bytes) lo = mid;
                else hi = mid - 1;
            }
            return lo;
        };
        int64_t lo = largest(true);
        if (lo == 0) lo = largest(false);
        if (lo == 0) {
            set_error("fk_lloyd_ooc: dev_ws of %zu bytes cannot hold even a 1024-row chunk", dev_ws_bytes);
            return FK_EWORKSPACE;
        }
        chunk_rows = lo * unit < N ? lo * unit : N;
    }
    if (chunk_rows > N) chunk_rows = N;
    if (!ooc_layout(chunk_rows, d, K, t, &L, &gfull)) {
        set_error("fk_lloyd_ooc: unsupported shape chunk_rows=%lld d=%d K=%d", (long long)chunk_rows, d, K);
        return FK_EUNSUPPORTED;
    }
    if (L.total > dev_ws_bytes) {
        set_error("fk_lloyd_ooc: dev_ws too small: %zu bytes given, %zu needed for chunk_rows=%lld",
                  dev_ws_bytes, L.total, (long long)chunk_rows);
        return FK_EWORKSPACE;
    }
    if (iters == 0) return FK_OK;

    char* base = (char*)dev_ws;
    void* xbuf[2] = {base, base + L.chunk_bytes};
    void* core = base + 2 * L.chunk_bytes;
    int32_t* chunk_assign = (int32_t*)(base + 2 * L.chunk_bytes + L.core_bytes);
    const Workspace wfull = carve(gfull, core, false);
    const bool early = L.with_late <= dev_ws_bytes;
    float* const late_sums = (float*)(base + L.total);
    int32_t* const late_counts = (int32_t*)(base + L.total + align_up(2 * L.late_sum_bytes, 256));
    const size_t row_bytes = (size_t)d * elem_size(t);                 // a row on the host
    const size_t dev_row_bytes = (size_t)gfull.d * elem_size(t);       // a padded row in a chunk buffer
    // Rows arrive as they are stored and the kernels read them so: a pitched copy moves a row at a
    // time (143690 rows of 25 bf16 values, one iteration: 1144 ms against 0.43 with the plain copy).
    const bool pad = gfull.d != gfull.d_user && gfull.d_user < 8;
    if (!pad) gfull.len = gfull.d_user;
    const int64_t nchunks = cdiv(N, chunk_rows);
    float* const C_user = C_f32;

    hipStream_t cs = (hipStream_t)stream;
    // Copies beside the kernels need a stream and events: some 95 us to make and to give back, and waits
    // in every chunk.  One chunk has nothing to be copied beside; and where all copies of the call are a
    // few MiB they take less than that: they go to the caller's stream, read by a kernel, which starts
    // sooner than a copy engine.  us, beside / so: 1000 points, d = 32, K = 8 120 / 38; 24533, d = 32,
    // K = 13 in three chunks 209 / 114, in eight 360 / 158; 2230 fp32, d = 512, K = 16, two iterations of
    // eight, 9 MiB 763 / 649; 16000, d = 256, K = 100, 8 MiB 312 / 280; 40000, d = 200, K = 100, 15 MiB
    // 511 / 505; 200000, d = 64 in one chunk, 24 MiB by the copy engine 595 / 532.
    const size_t copied = (size_t)N * row_bytes * (size_t)(nchunks == 1 ? 1 : iters);
    // The kernel reads what it is told to.  Both ends of X_host are pinned, but they may be the ends of two allocations with
    // anything between them, or of memory that another device has mapped: those go to a copy, which the runtime checks.
    void* X_dev = nullptr;
    if (!pad && copied <= ((size_t)16 << 20) && pinned_here) {
        hipDeviceptr_t base = nullptr;
        size_t size = 0;
        if (hipHostGetDevicePointer(&X_dev, (void*)X_host, 0) != hipSuccess ||
            hipMemGetAddressRange(&base, &size, (hipDeviceptr_t)X_dev) != hipSuccess ||
            !lies_within(X_dev, (size_t)N * row_bytes, base, size)) {
            (void)hipGetLastError();
            X_dev = nullptr;
        }
    }
    const bool beside = !X_dev && (pad || nchunks > 1);
    hipStream_t side = nullptr;
    hipEvent_t ready[2] = {nullptr, nullptr}, freed[2] = {nullptr, nullptr};
    fk_status st = FK_OK;
    auto cleanup = [&]() {
        for (int i = 0; i < 2; ++i) {
            if (ready[i]) (void)hipEventDestroy(ready[i]);
            if (freed[i]) (void)hipEventDestroy(freed[i]);
        }
        if (side) (void)hipStreamDestroy(side);
    };
#define OOC_HIP(call)                                      \
    do {                                                   \
        hipError_t _e = (call);                            \
        if (_e != hipSuccess) {                            \
            st = hip_fail(_e, #call);                      \
            (void)hipDeviceSynchronize();                  \
            cleanup();                                     \
            return st;                                     \
        }                                                  \
    } while (0)
#define OOC_TRY(expr)                                      \
    do {                                                   \
        st = (expr);                                       \
        if (st != FK_OK) {                                 \
            (void)hipDeviceSynchronize();                  \
            cleanup();                                     \
            return st;                                     \
        }                                                  \
    } while (0)

    if (beside) OOC_HIP(hipStreamCreateWithFlags(&side, hipStreamNonBlocking));
    for (int i = 0; beside && i < 2; ++i) {
        OOC_HIP(hipEventCreateWithFlags(&ready[i], hipEventDisableTiming));
        OOC_HIP(hipEventCreateWithFlags(&freed[i], hipEventDisableTiming));
    }
    bool used[2] = {false, false};
    int64_t held[2] = {-1, -1};                  // chunk in each buffer
    if (pad) {
        OOC_HIP(hipMemsetAsync(xbuf[0], 0, 2 * L.chunk_bytes, side));
        OOC_TRY(launch_copy_rows(C_user, wfull.c_pad_f32, K, gfull.d_user, gfull.d, 4, cs));
        C_f32 = wfull.c_pad_f32;
    }

    for (int it = 0; it < iters; ++it) {
        OOC_TRY(launch_round_centroids(gfull, C_f32, t == FK_F32 ? nullptr : wfull.c_lp,
                                       wfull.c_frag, wfull.c_bias, cs));
        // the chunks [first, first + count) are in the buffers and taken before their turn, the one whose
        // buffer chunk 0 goes to (the even one) first
        int64_t first = 0, count = 0;
        if (early && it > 0 && nchunks > 2) {
            first = held[0] < held[1] ? held[0] : held[1];
            count = first > 0 && held[0] + held[1] == 2 * first + 1 ? 2 : 0;
        }
        for (int64_t at = 0; at < nchunks; ++at) {
            const bool waits = at < count;       // its sums wait for their turn
            const int64_t c = waits ? held[at] : at - count < first || count == 0 ? at - count : at;
            const int bi = (int)(c & 1);
            const int64_t r0 = c * chunk_rows;
            const int64_t rows = (N - r0) < chunk_rows ? (N - r0) : chunk_rows;
            if (held[bi] != c) {
                // side stream: refill buffer bi once its previous consumer is done
                if (beside && used[bi]) OOC_HIP(hipStreamWaitEvent(side, freed[bi], 0));
                if (X_dev)
                    OOC_TRY(launch_copy_bytes((const char*)X_dev + (size_t)r0 * row_bytes, xbuf[bi], (size_t)rows * row_bytes, cs));
                else if (pad)
                    OOC_HIP(hipMemcpy2DAsync(xbuf[bi], dev_row_bytes, (const char*)X_host + (size_t)r0 * row_bytes,
                                             row_bytes, row_bytes, (size_t)rows, hipMemcpyHostToDevice, side));
                else
                    OOC_HIP(hipMemcpyAsync(xbuf[bi], (const char*)X_host + (size_t)r0 * row_bytes,
                                           (size_t)rows * row_bytes, hipMemcpyHostToDevice, beside ? side : cs));
                if (beside) OOC_HIP(hipEventRecord(ready[bi], side));
                held[bi] = c;
            }
            // compute stream
            if (beside) OOC_HIP(hipStreamWaitEvent(cs, ready[bi], 0));
            // A shorter tail chunk keeps the full chunk's tiling parameters and buffers
            // (every buffer is sized for chunk_rows); only the row-dependent counts shrink.
            Geometry g = gfull;
            const Workspace& w = wfull;
            g.N = rows;
            g.sort_blocks = (int)cdiv(rows, g.sort_tile);
            g.max_items = rows / g.rows_per_item + K;
            int32_t* a = assign ? assign + r0 : chunk_assign;
            if (t == FK_F32)
                OOC_TRY(launch_assign(g, xbuf[bi], C_f32, nullptr, a, nullptr, cs, &w));
            else
                OOC_TRY(launch_assign(g, xbuf[bi], w.c_frag, w.c_bias, a, nullptr, cs));
            FinalizeArgs fa;
            fa.C_prev_f32 = C_f32;
            fa.C_out_f32 = C_f32;
            fa.C_out_lp = nullptr;
            fa.c_frag = nullptr;
            fa.c_bias = nullptr;
            fa.counts = waits ? late_counts + (c - first) * K : counts;
            fa.sums = waits ? late_sums + (c - first) * K * gfull.d : wfull.sums;
            fa.accumulate = !waits && c > 0;
            fa.normalise = (at + 1 == nchunks);
            if (count > 0 && c == first - 1) {
                fa.late_sums = late_sums;
                fa.late_counts = late_counts;
                fa.late = (int)count;
            }
            if (g.gather_parts > 0) {
                OOC_TRY(launch_gather_update(g, w, xbuf[bi], a, fa, cs));
                g.max_items = (int64_t)K * g.gather_parts;
                if (gather_needs_merge(g, fa))
                    OOC_TRY(launch_finalize(g, w, nullptr, nullptr, fa, cs, w.gather_counts, g.gather_parts));
            } else {
                OOC_TRY(launch_sort_inverse(g, w, a, w.sorted_idx, w.seg_off, w.item_off, cs));
                OOC_TRY(launch_segment_reduce(g, w, xbuf[bi], w.sorted_idx, w.seg_off, w.item_off, cs));
                OOC_TRY(launch_finalize(g, w, w.seg_off, w.item_off, fa, cs));
            }
            if (beside) OOC_HIP(hipEventRecord(freed[bi], cs));
            used[bi] = true;
        }
    }
    if (pad) OOC_TRY(launch_copy_rows(C_f32, C_user, K, gfull.d, gfull.d_user, 4, cs));
    if (beside) OOC_HIP(hipStreamSynchronize(side));
    OOC_HIP(hipStreamSynchronize(cs));
    cleanup();
    return FK_OK;
#undef OOC_HIP
#undef OOC_TRY
}

}  // extern "C"
