// Driver for tests/test_host_decisions.py: what the library decides on the host before it launches anything,
// asked of the functions that decide it.  No kernel is launched and no GPU is needed.
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

int main() {
    if (option_is_read_once()) return 1;
    printf("host decisions ok\n");
    return 0;
}
