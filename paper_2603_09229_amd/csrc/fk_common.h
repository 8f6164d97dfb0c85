// Internal declarations shared by the flashkm translation units (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>

#include "flashkm.h"

namespace fk {

// ---------------------------------------------------------------- errors
void set_error(const char* fmt, ...);
fk_status hip_fail(hipError_t e, const char* what);

#define FK_HIP(call)                                           \
    do {                                                       \
        hipError_t _e = (call);                                \
        if (_e != hipSuccess) return fk::hip_fail(_e, #call);  \
    } while (0)

#define FK_TRY(expr)                       \
    do {                                   \
        fk_status _s = (expr);             \
        if (_s != FK_OK) return _s;        \
    } while (0)

// ---------------------------------------------------------------- small helpers
constexpr int kWave = 64;

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
// Whether `bytes` bytes from `at` on all lie in the allocation of `size` bytes at `base`.
inline bool lies_within(const void* at, size_t bytes, const void* base, size_t size) {
    const uintptr_t a = (uintptr_t)at, b = (uintptr_t)base;
    return a >= b && a - b <= size && bytes <= size - (a - b);
}
inline size_t elem_size(fk_dtype t) { return t == FK_F32 ? 4 : 2; }
// What the host-side choices need to know about the current device, asked of the runtime once
// per device: compute units, LDS per compute unit, and the size of the last-level cache (the
// largest cache the HSA runtime lists for the agent; the L2 size HIP reports if that fails).
// With no GPU in the process: 256 units, 160 KiB, 256 MiB (MI355X).
struct DeviceInfo {
    int cus;
    int64_t lds_bytes;
    int64_t llc_bytes;
};
constexpr int kMaxDevices = 64;
int current_device();                 // ordinal of the current HIP device, 0 if there is none
const DeviceInfo& device_info();
inline int device_cu_count() { return device_info().cus; }

// A value remembered per device (kernel attributes set, occupancy queried): 0 = not yet known.
// Racing first calls compute the same value twice, which is harmless.
struct PerDeviceInt {
    std::atomic<int> v[kMaxDevices];
    int get() const { return v[current_device()].load(std::memory_order_relaxed); }
    void set(int x) { v[current_device()].store(x, std::memory_order_relaxed); }
};

// ---------------------------------------------------------------- problem geometry
//
// Centroids for the MFMA path are kept in "fragment order": centroid tile (32 rows) x
// feature chunk (16 features) x lane (64) x 8 elements, so that a 32x32x16 MFMA A-operand
// is one 16-byte LDS read per lane at lane*16.  Rows beyond K and features beyond d are
// zero; their score bias is -inf so they never win.
struct Geometry {
    int B;
    int64_t N;        // points per instance
    int d, K;         // d: row width the kernels see (a multiple of 8)
    int d_user;       // row width of the caller's arrays
    int len;          // elements of a row of X and C as the kernels are given them: d_user where they
                      // read the caller's rows (row_piece16 / row_piece32), d after the rows have
                      // been copied into zero-padded ones (zeros change no distance and no mean)
    fk_dtype t;
    int dchunks;      // 16-feature chunks of the assignment kernel: ceil(d / 16) or the next number it is compiled for
    int ktiles;       // ceil(K / 32)
    bool one_pass;    // the one-pass updates may be taken: the process-wide option as it stood when this
                      // was filled in.  A call asks it once: whether rows are padded and which kernel
                      // reads them must follow from one answer (the kernel for few clusters reads rows
                      // of width d, past the end of X where they were not padded)
    int f32_filter;   // the option of the filtered fp32 assignment, likewise: an update writes the split centroids of
                      // the next assignment only if the one before it has laid them out
    // counting sort
    int sort_bits;    // bits of a cluster id, ceil(log2 K), >= 1
    int sort_passes;  // 1 when K <= 2048, else 2
    int pass_bits[2];
    int sort_tile;    // keys per sort workgroup
    int sort_blocks;  // workgroups per instance = ceil(N / sort_tile)
    // segment reduction
    int rows_per_item;   // R: sorted positions reduced into one partial row
    int waves_per_item;  // 1, or 4 (a whole workgroup) for the long items of few-cluster shapes
    int64_t max_items;   // upper bound on sum_k ceil(n_k / R) per instance
    // sort-free update for few clusters (16-bit storage, K <= 32, d <= 128): most workgroups
    // per instance it may use, 0 when the shape is not eligible
    int fused_grid_cap;
    // one-pass update with the K x d table split over the registers of a workgroup (16-bit
    // storage, 32 < K <= 256, d <= 128): most workgroups per instance, 0 when not eligible
    int table_grid_cap;
    // one-pass assignment + sums for small fp32 problems (K <= 64, d <= 128, at most 2^17 points
    // in all; see fk_f32_fused.hip): most workgroups per instance, 0 when not eligible
    int f32_grid_cap;
    // small instances: the update without a sort (see gather_update_kernel in fk_update.hip): into how many
    // parts an instance is cut, 0 when the shape is not eligible
    int gather_parts;
};

// Carved device workspace (all pointers 256-byte aligned inside the caller's buffer).
struct Workspace {
    void* c_lp;          // [B,K,d] low-precision centroids consumed by assign (lloyd only)
    void* c_frag;        // [B,ktiles,dchunks,64,8] fragment-ordered centroids (16-bit types);
                         // FK_F32: [B,ktiles,2*dchunks+1,64,8], see fk_f32_filter.hip
    float* c_bias;       // [B,ktiles*32] -||c||^2/2, -inf for padding rows (FK_F32: squared norms)
    int32_t* sorted_idx; // [B,N]
    int32_t* seg_off;    // [B,K+1]
    int32_t* item_off;   // [B,K+1] exclusive scan of ceil(n_k / R)
    int32_t* block_hist; // [B,bins,sort_blocks] per-workgroup digit histograms
    int32_t* digit_off;  // [B,2048+1] digit offsets of the current radix pass
    uint16_t* keys_tmp;  // [B,N] keys after pass 1 (two-pass sort only)
    int32_t* vals_tmp;   // [B,N] values after pass 1 (two-pass sort only)
    uint16_t* keys_sorted;// [B,N] sorted keys (two-pass sort only)
    float* partial;      // [B,max(max_items, K*(largest one-pass grid cap)),d] per-item segment sums
    int32_t* wg_counts;  // [B,K,grid cap] per-workgroup counts (one-pass updates only)
    int32_t* gather_counts;  // [B,K,gather_parts] the same of an update without a sort
    float* sums;         // [B,K,d] accumulated sums (chunked mode)
    float* f32_shift;    // [B,dchunks*16] shift of the filtered fp32 assignment (fk_f32_filter.hip)
    int32_t* f32_list_len; // [B] points it has left open (the points themselves: sorted_idx)
    int32_t* f32_pair_len; // [B] those of them that are open between two centroids; memory that the update in use does not read
                           // while it clears this for the next assignment: an update without a sort has no segments, one that
                           // sorts is done with its totals
    void* x_pad;         // [B,N,d] zero-padded copy of X            (only when needs_padded_rows)
    float* c_pad_f32;    // [B,K,d] zero-padded fp32 centroids       (likewise)
    void* c_pad_lp;      // [B,K,d] zero-padded centroids, dtype t   (likewise)
    size_t bytes;        // total bytes carved
};

// Shapes whose rows are copied into zero-padded ones first: the one-pass update for few clusters
// copies whole 16-byte pieces straight to LDS, and rows of fewer than 8 elements hold no piece.
inline bool needs_padded_rows(const Geometry& g) { return g.d != g.d_user && (g.d_user < 8 || g.fused_grid_cap > 0); }

bool make_geometry(int B, int64_t N, int d, int K, fk_dtype t, Geometry* g);
// Lays the workspace out from `base` (may be NULL to only compute the size).  padded_x = false
// leaves out the zero-padded copy of X (the out-of-core call pads through its pitched copies).
Workspace carve(const Geometry& g, void* base, bool padded_x = true);

// ---------------------------------------------------------------- kernel launchers
// Each enqueues on `s` and returns FK_OK / FK_EHIP.  Pointers are device pointers.

// C (dtype t, [B,K,d]) -> fragment-ordered copy + score bias.  16-bit types only.
fk_status launch_prepare_centroids(const Geometry& g, const void* C_lp, void* c_frag,
                                   float* c_bias, hipStream_t s);
// C_f32 -> C_lp (round to nearest even), and for 16-bit types also c_frag / c_bias.
fk_status launch_round_centroids(const Geometry& g, const float* C_f32, void* C_lp,
                                 void* c_frag, float* c_bias, hipStream_t s);
// Fused distance + online argmin.  16-bit: reads c_frag/c_bias; fp32: reads C directly.
// fp32 with a workspace may take the filtered form (fk_f32_filter.hip), which uses the centroid
// buffers and sorted_idx of it; without one (nullptr) the direct kernels.
enum class F32Split {
    kAmongCentroids,     // laid out by the assignment, shifted by a mean of the centroids
    kAmongPoints,        // by a mean of the points: the first assignment of a fit
    kWritten             // the last update has written them, with the shift of the first assignment, and cleared the lists (FinalizeArgs)
};
fk_status launch_assign(const Geometry& g, const void* X, const void* C_or_frag,
                        const float* c_bias, int32_t* assign, float* min_dist, hipStream_t s,
                        const Workspace* w = nullptr, F32Split split = F32Split::kAmongCentroids);
// fp32: candidates from split bf16 products on the matrix cores, the open points by direct differences
fk_status launch_f32_filter(const Geometry& g, const Workspace& w, const float* X, const float* C,
                            int32_t* assign, float* min_dist, F32Split split, hipStream_t s);
bool f32_filter_enabled(const Geometry& g);
int f32_filter_option();
// Which of N points a fit's shift is taken from: the fractional parts of multiples of the golden ratio, spread evenly and met by no
// period of the data.
__host__ __device__ inline uint32_t sampled_row(uint32_t i, uint32_t N) { return (uint32_t)((uint64_t)(i * 0x9E3779B9u) * N >> 32); }
// Half workgroups (of 256 threads) that measure distances, `lanes` threads a point.  A launch dimension holds fewer
// than 2^32 threads, which one point per group of 16 lanes reaches at 2^28 points.
inline int64_t f32_distance_blocks(int64_t N, int lanes) {
    const int64_t groups = cdiv(N, 256 / lanes), most = (int64_t)1 << 20;
    return groups < most ? groups : most;
}
// direct kernels, d <= 128: the four waves of a workgroup share a centroid tile (few points)
inline bool f32_direct_is_split(const Geometry& g) { return g.d <= 128 && (int64_t)g.B * g.N < ((int64_t)1 << 18); }
void set_f32_filter_option(int v);         // -1 = by shape, 0 = never, 1 = always
// Tile shape the sweeping assign kernel would use for this problem (see fk_assign.hip).
int choose_assign_variant(const Geometry& g);
void set_assign_variant_override(int v);   // -1 = choose from the shape
// Few centroids: persistent streaming kernel instead of the sweeping one (see fk_assign.hip).
bool assign_uses_stream_kernel(const Geometry& g);
void set_assign_stream_option(int v);      // -1 = by shape, 0 = never, 1 = whenever eligible
int wide_kernel_waves(const Geometry& g);  // of the kernel for rows of more than 128 features
// Few points: the waves of a workgroup share the centroid tiles of 32 or 64 points (see fk_assign.hip).
bool assign_uses_few_kernel(const Geometry& g);
void set_assign_few_option(int v);         // -1 = by shape, 0 = never, 1..4 = one of its forms
// ... straight from C [B,K,d] of dtype t, without launch_prepare_centroids
bool assign_few_takes_rows(const Geometry& g);
fk_status launch_assign_rows(const Geometry& g, const void* X, const void* C, int32_t* assign,
                             float* min_dist, hipStream_t s);
// Stable argsort by cluster id -> sorted_idx, seg_off (+ item_off when w.item_off != NULL).
fk_status launch_sort_inverse(const Geometry& g, const Workspace& w, const int32_t* assign,
                              int32_t* sorted_idx, int32_t* seg_off, int32_t* item_off,
                              hipStream_t s);
// Whether the scatter kernel adds the workgroups' histograms up itself instead of a scan kernel doing it.  It
// saves the launch and costs a thread per bin one read of every workgroup's count, one after the other.
// fk_sort_inverse, us with the scan and without:
//   64 bins, workgroups  8: 15.6 12.7   32: 15.6 13.8   48: 15.6 14.2   64: 15.7 14.9   512: 21.8 36.0
//   16 bins             64: 13.8 13.6   80: 13.9 14.4
// Where the workgroups come in several rounds each of them pays, and few bins gain least:
//   16 bins, 16 instances of 48: 19.8 18.8, of 64: 26.9 27.4; 64 of 24: 34.7 32.6, of 48: 63.5 65.7
//   256 bins, 64 instances of 48: 80.2 76.2, 300 of 32: 243 230, of 48: 409 411
// Many bins times many workgroups: 1000 bins, 32: 18.6 17.7; 2^16 counts 42.0 44.2 (fk_update).
inline bool sort_scatter_scans(int instances, int blocks, int bins) {
    const int64_t all = (int64_t)instances * blocks;
    const int most = all <= 512 ? 64 : all <= 1024 || bins >= 256 ? 48 : 24;
    return blocks > 1 && blocks <= most && bins <= 1024 && blocks * bins <= 32768;
}
// Largest bin count for which the scatter stages its tile through LDS (-1 = the built-in 1024).
void set_sort_stage_bins(int v);
// Per-item segment sums of gathered rows -> w.partial.
fk_status launch_segment_reduce(const Geometry& g, const Workspace& w, const void* X,
                                const int32_t* sorted_idx, const int32_t* seg_off,
                                const int32_t* item_off, hipStream_t s);
// Merge item sums per cluster; optionally accumulate into sums/counts; optionally
// normalise and emit centroids (fp32 master, rounded copy, fragment copy, bias).
struct FinalizeArgs {
    const float* C_prev_f32;
    float* C_out_f32;
    void* C_out_lp;      // may be NULL
    void* c_frag;        // may be NULL
    float* c_bias;       // may be NULL
    int32_t* counts;     // [B,K]
    float* sums;         // [B,K,d] (needed when accumulate || !normalise)
    bool accumulate;     // add onto sums / counts already there
    const float* late_sums = nullptr;      // [late][B,K,d], [late][B,K]: parts to add after these ones,
    const int32_t* late_counts = nullptr;  // one after the other
    int late = 0;
    bool normalise;      // divide and write centroids
    // fp32, filtered assignment next: its split centroids, which the first assignment of the call has laid out (NULL: not wanted)
    void* c_split = nullptr;
    const float* shift = nullptr;
    float* c2 = nullptr;
    int32_t *list_len = nullptr, *pair_len = nullptr;
};
// With wg_counts (few-cluster path) cluster k owns partial rows [k*G, (k+1)*G) and the counts
// wg_counts[b][k][0..G) instead of what seg_off / item_off say (those may then be NULL).
fk_status launch_finalize(const Geometry& g, const Workspace& w, const int32_t* seg_off,
                          const int32_t* item_off, const FinalizeArgs& a, hipStream_t s,
                          const int32_t* wg_counts = nullptr, int wg_per_cluster = 0);

// Small instances (g.gather_parts > 0): every workgroup reads all assignments of its part of the instance and adds the rows
// of one cluster.  Writes what launch_finalize does; where gather_needs_merge, w.partial / w.gather_counts as
// launch_stream_update with wg_per_cluster = g.gather_parts instead.
fk_status launch_gather_update(const Geometry& g, const Workspace& w, const void* X, const int32_t* assign,
                               const FinalizeArgs& a, hipStream_t s);
// (parts that wait for their turn are added by the merge kernel)
inline bool gather_needs_merge(const Geometry& g, const FinalizeArgs& a) { return g.gather_parts > 1 || a.late > 0; }
bool limit_gather_parts(Geometry* g);      // to the partial rows that the sorted update has room for; whether that changed them
int choose_gather_parts(int B, int64_t N, int d, int K, fk_dtype t);
void set_gather_update_option(int v);      // -1 = by shape, 0 = never, 1..64 = always, in that many parts

// Few clusters: stream X once, add every 32-point batch into per-workgroup K x d tables with a
// one-hot MFMA (no sort, no gather); with compute_assign the assignment is computed (and, where
// keep_assign says so, written) in the same pass, otherwise read.  Leaves w.partial / w.wg_counts ready for
// launch_finalize with max_items = K * (*grid_out) and wg_per_cluster = *grid_out.
fk_status launch_stream_update(const Geometry& g, const Workspace& w, const void* X,
                               int32_t* assign, bool compute_assign, bool keep_assign, int* grid_out,
                               hipStream_t s);
inline bool fused_update_enabled(const Geometry& g) { return g.fused_grid_cap > 0 && g.one_pass; }
void set_fused_update_option(int v);       // 0 = never, otherwise whenever the shape allows
bool fused_update_allowed();               // the option above is not 0

// Up to 256 clusters: assignment and sums in one pass over X with the table of sums in the
// registers of a persistent workgroup (see fk_table.hip).  Computes and writes the assignment;
// leaves w.partial / w.wg_counts as launch_stream_update does.
fk_status launch_table_update(const Geometry& g, const Workspace& w, const void* X,
                              int32_t* assign, int* grid_out, hipStream_t s);
inline bool table_update_enabled(const Geometry& g) { return g.table_grid_cap > 0 && g.one_pass; }

// Small fp32 problems, up to 64 clusters: assignment and sums in one pass over X (see
// fk_f32_fused.hip).  C_f32 [B,K,d] are the centroids to assign against.  Computes and writes the
// assignment; leaves w.partial / w.wg_counts as launch_stream_update does.
fk_status launch_f32_update(const Geometry& g, const Workspace& w, const void* X,
                            const float* C_f32, int32_t* assign, int* grid_out, hipStream_t s);
inline bool f32_update_enabled(const Geometry& g) { return g.f32_grid_cap > 0 && g.one_pass; }

// Row re-layout for widths that are not a multiple of 8: dst[r][j] = j < d_src ? src[r][j] : 0
// for j < d_dst (padding, d_dst > d_src) or dst[r][j] = src[r][j] for j < d_dst (un-padding,
// d_dst < d_src).  elem = bytes per element (2 or 4).
fk_status launch_copy_rows(const void* src, void* dst, int64_t rows, int d_src, int d_dst,
                           int elem, hipStream_t s);

// Comparator: the standard implementation (paper Algorithm 1); see fk_standard.hip.
fk_status launch_standard_assign(const Geometry& g, const Workspace& w, const void* X,
                                 const void* C_lp, float* D, int32_t* assign, hipStream_t s);
fk_status launch_standard_update(const Geometry& g, const void* X, const int32_t* assign,
                                 const float* C_prev, float* C_out, int32_t* counts, float* sums,
                                 hipStream_t s);

}  // namespace fk
