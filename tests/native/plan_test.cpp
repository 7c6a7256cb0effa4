// Test driver of the cut of a batch (paper_2003_09956_amd/csrc/batch_plan.hpp).
// No device is needed.  Exits non-zero on the first failed check.
#include <cstdio>

#include "batch_plan.hpp"

static int failures = 0;
#define EXPECT(cond)                                                                          \
    do {                                                                                      \
        if (!(cond)) {                                                                        \
            std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #cond);     \
            ++failures;                                                                       \
        }                                                                                     \
    } while (0)

using namespace modap_host;

// Whether `count` systems of m rows of ldA elements are swept by groups.
// other_group: bytes of the largest group of another system.
static bool by_groups(int64_t count, int64_t m, int64_t ldA, int64_t es, int32_t item_kib, int64_t per_cu,
                      int64_t other_group = 0) {
    const BatchCut cut = plan_cut(m, ldA, es, item_kib, 0, 16, 8);
    const int64_t bytes = m * ldA * es, group = cut.cells * cut.rows_per_cell * ldA * es;
    return cut.cells > 1 &&
           plan_cells_per_item(cut, ldA * es, count * bytes, 256 * per_cu, 256, std::max(group, other_group)) == cut.cells;
}

int main() {
    // a part of any system is between a cell and a group
    for (int64_t es : {2, 4, 8})
        for (int64_t ldA : {64, 256, 1000, 2000, 4000})
            for (int64_t m : {1, 100, 3000, 40000})
                for (int64_t total : {int64_t(1), m * ldA * es, 100 * m * ldA * es, int64_t(1) << 40}) {
                    const BatchCut cut = plan_cut(m, ldA, es, 4096, 0, 16, 8);
                    EXPECT(cut.cells >= 1 && cut.cells <= 8 && cut.rows_per_cell % 16 == 0);
                    const int64_t group = cut.cells * cut.rows_per_cell * ldA * es;
                    for (int64_t largest : {group, 100 * group}) {
                        const int64_t c = plan_cells_per_item(cut, ldA * es, total, 512, 256, largest);
                        EXPECT(c >= 1 && c <= cut.cells);
                    }
                }
    // 7/4 groups a CU and more: eight groups a system here
    EXPECT(by_groups(64, 3000, 1400, 4, 8192, 2));     // 2.0 groups a CU
    EXPECT(by_groups(128, 3000, 1400, 4, 8192, 2));
    EXPECT(by_groups(64, 3000, 700, 8, 8192, 2));
    EXPECT(by_groups(128, 3000, 600, 4, 4096, 2));
    EXPECT(by_groups(64, 4000, 2000, 2, 4096, 1));
    // beside larger groups: less than half the share of a workgroup
    EXPECT(!by_groups(64, 3000, 1400, 4, 8192, 2, int64_t(8) << 20));
    EXPECT(by_groups(300, 3000, 1400, 4, 8192, 2, int64_t(32) << 20));
    EXPECT(!by_groups(48, 3000, 1400, 4, 8192, 2));    // 1.5
    EXPECT(!by_groups(32, 4000, 2000, 2, 4096, 1));    // 1.0
    EXPECT(!by_groups(7, 4000, 2000, 2, 4096, 1));
    // the grid: two workgroups a CU from two items each on, one below, where the
    // count of items is not set; a tuned grid as it is; never more than items
    EXPECT(plan_grid(0, 2, 256, 1024, 0) == 512);
    EXPECT(plan_grid(0, 2, 256, 1023, 0) == 256);
    EXPECT(plan_grid(0, 2, 256, 1023, 1) == 512);
    EXPECT(plan_grid(0, 2, 256, 512, 1) == 512);
    EXPECT(plan_grid(0, 2, 256, 100, 1) == 100);
    EXPECT(plan_grid(0, 1, 256, 300, 0) == 256);
    EXPECT(plan_grid(0, 2, 256, 100, 0) == 100);
    EXPECT(plan_grid(0, 2, 256, 0, 0) == 1);
    EXPECT(plan_grid(512, 2, 256, 600, 0) == 512);
    EXPECT(plan_grid(300, 2, 256, 200, 4) == 200);
    if (failures) return 1;
    std::puts("all plan checks passed");
    return 0;
}
