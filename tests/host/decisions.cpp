// Driver for tests/test_host_decisions.py: what the library decides on the host before it launches anything,
// asked of the functions that decide it.  No kernel is launched and no GPU is needed.
#include <stdint.h>
#include <stdio.h>

#include "fk_common.h"
#include "flashkm.h"

#define CHECK(c) do { if (!(c)) { fprintf(stderr, "CHECK failed line %d: %s\n", __LINE__, #c); return 1; } } while (0)

// One call takes the process-wide option once: a thread that changes it meanwhile must not leave rows
// unpadded for a kernel that reads padded ones (or any other half of either choice).
static int option_is_read_once() {
    struct { fk_dtype t; int64_t N; int d, K; } shapes[] = {
        {FK_F16, 1000, 12, 16}, {FK_BF16, 100000, 100, 32}, {FK_F16, 5000, 33, 100}, {FK_F32, 3000, 50, 20}, {FK_F16, 100, 5, 4},
    };
    for (auto& s : shapes)
        for (int before : {0, -1}) {
            fk::Geometry g;
            CHECK(fk_set_option("fused_update", before) == FK_OK);
            CHECK(fk::make_geometry(1, s.N, s.d, s.K, s.t, &g));
            const bool taken[3] = {fk::fused_update_enabled(g), fk::table_update_enabled(g), fk::f32_update_enabled(g)};
            CHECK((taken[0] || taken[1] || taken[2]) == (before != 0));
            CHECK(fk_set_option("fused_update", before ? 0 : -1) == FK_OK);
            CHECK(fk::fused_update_enabled(g) == taken[0] && fk::table_update_enabled(g) == taken[1] && fk::f32_update_enabled(g) == taken[2]);
        }
    return fk_set_option("fused_update", -1) == FK_OK ? 0 : 1;
}

// The same for the filtered fp32 assignment: an update that writes what the next assignment multiplies rests on the assignment
// before it having laid that out.
static int filter_is_chosen_once() {
    struct { int64_t N; int d, K; bool by_shape; } shapes[] = {
        {300000, 96, 400, true}, {5000, 256, 40, true}, {1000, 32, 4, false}, {2000, 1, 918, false}, {100000, 7, 200, false},
    };
    for (auto& s : shapes)
        for (int before : {-1, 0, 1})
            for (int after : {-1, 0, 1}) {
                fk::Geometry g;
                CHECK(fk_set_option("assign_f32_filter", before) == FK_OK);
                CHECK(fk::make_geometry(1, s.N, s.d, s.K, FK_F32, &g));
                CHECK(fk_set_option("assign_f32_filter", after) == FK_OK);
                CHECK(fk::f32_filter_enabled(g) == (before < 0 ? s.by_shape : before == 1));
                fk::Geometry part = g;               // a chunk of an out-of-core call
                part.N = s.N / 3;
                CHECK(before < 0 || fk::f32_filter_enabled(part) == (before == 1));
            }
    return fk_set_option("assign_f32_filter", -1) == FK_OK ? 0 : 1;
}

// A fit keeps one shift, a mean of some of 32 of its points: they lie in X, in every sixteenth of it, and where the clusters take turns in rows of
// data no more than a quarter of them belong to one of eight or more.
static int shifts_lie_among_points() {
    for (uint32_t N : {1u, 2u, 31u, 32u, 1000u, 65536u, 1u << 20, 16777217u, 0x7FFFFFFFu}) {
        bool met[16] = {};
        for (uint32_t i = 0; i < 32; ++i) {
            const uint32_t row = fk::sampled_row(i, N);
            CHECK(row < N);
            met[(uint64_t)row * 16 / N] = true;
        }
        for (bool m : met) CHECK(m || N < 32);
        for (uint32_t clusters : {8u, 64u, 256u, 1000u, 1024u, 4096u}) {
            int most = 0;
            for (uint32_t i = 0; i < 32; ++i) {
                int same = 0;
                for (uint32_t j = 0; j < 32; ++j) same += fk::sampled_row(i, N) % clusters == fk::sampled_row(j, N) % clusters;
                most = same > most ? same : most;
            }
            CHECK(most <= 8 || N < 1000);
        }
    }
    return 0;
}

// A launch dimension holds fewer than 2^32 threads.
static int launches_fit() {
    for (int lanes : {4, 8, 16})
        for (int64_t N : {(int64_t)1, (int64_t)16, (int64_t)17, (int64_t)1 << 24, ((int64_t)1 << 28) - 16, (int64_t)1 << 28, ((int64_t)1 << 31) - 1}) {
            const int64_t blocks = fk::f32_distance_blocks(N, lanes);
            CHECK(blocks >= 1 && blocks * 256 <= UINT32_MAX);
            CHECK(N > ((int64_t)1 << 24) || blocks * (256 / lanes) >= N);   // one group each where that fits
        }
    for (int option : {-1, 1})
        for (int64_t below : {1, 255, 256, 257}) {
            fk::Geometry g;
            CHECK(fk_set_option("assign_f32_filter", option) == FK_OK);
            CHECK(fk::make_geometry(1, ((int64_t)1 << 31) - below, 8, 64, FK_F32, &g));
            CHECK(fk::f32_filter_enabled(g) == (below >= 256));
            CHECK(!fk::f32_filter_enabled(g) || fk::cdiv(g.N, 256) * 512 <= UINT32_MAX);
        }
    return fk_set_option("assign_f32_filter", -1) == FK_OK ? 0 : 1;
}

// The scatter reads one count per workgroup and bin, in a row: only ever few of them, whatever the bins.
static int few_counts_in_a_row() {
    for (int instances : {1, 3, 64, 65535})
        for (int bins : {1, 2, 8, 64, 256, 1000, 1024, 1025, 2048})
            for (int blocks : {1, 2, 18, 32, 48, 64, 65, 128, 512, 4096, 65536}) {
                const bool scans = fk::sort_scatter_scans(instances, blocks, bins);
                CHECK(!scans || (blocks <= 64 && (int64_t)blocks * bins <= 32768));
                CHECK(scans || blocks < 2 || blocks > (instances > 3 ? 18 : 32) || bins > 1000);   // ... and all of those that gain
            }
    return 0;
}

// Host rows that a kernel reads lie in one allocation as a whole.
static int host_rows_lie_in_one_allocation() {
    const char* const base = (const char*)0x100000;
    const size_t size = 1 << 16;
    for (size_t off : {(size_t)0, (size_t)16, size - 16, size}) {
        const size_t left = size - off;
        CHECK(fk::lies_within(base + off, left, base, size) && fk::lies_within(base + off, 0, base, size));
        CHECK(!fk::lies_within(base + off, left + 1, base, size) && !fk::lies_within(base + off, SIZE_MAX, base, size));
        CHECK(!fk::lies_within(base + off, 2 * size, base, size));       // ... whose other end is in the next one
    }
    CHECK(!fk::lies_within(base - 16, 16, base, size) && !fk::lies_within(base - 16, 32, base, size));
    CHECK(!fk::lies_within(base + size + 16, 1, base, size) && !fk::lies_within(base, 1, nullptr, 0));
    return 0;
}

int main() {
    if (option_is_read_once() || filter_is_chosen_once() || shifts_lie_among_points() || launches_fit() || few_counts_in_a_row() || host_rows_lie_in_one_allocation()) return 1;
    printf("host decisions ok\n");
    return 0;
}
