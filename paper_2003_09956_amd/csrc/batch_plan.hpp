// How the batched sweep cuts each system into work items and which row form
// it runs for the system: the host-side decisions that fix what the batched
// sweep kernel reads, kept apart from the rest of the batch host code.
#pragma once

#include <algorithm>
#include <cstdint>

namespace modap_host {

// Row-length bucket of a system whose rows take C 16-byte chunks per lane of
// a wavefront (C = 1, 2, 4, 8).
inline int bucket_of(int C) { return C == 1 ? 0 : C == 2 ? 1 : C == 4 ? 2 : 3; }

// The cut of a system.  It depends on the system and the tile only, never on
// the other systems of the batch, so a system's results do not depend on them.
// The rows are cut into groups of about item_kib KiB of A, but into at least
// eight (min_items, if given) of at least kMinItemKib KiB; a group's partial
// of y is what the reduction adds up.  A group is cut into up to kGroupCells
// cells of at least cell_kib KiB (one, if min_items was given), whose partials
// are added in order -- by the sweep, where an item is a whole group, or by
// the reduction, where it is less: the same sums either way.  `unit` rows are
// the step that cells are a multiple of.  A cell's end costs the sweep ten rows
// of LDS traffic, so a cell has 256 KiB at least in 2 and 4 bytes an element (in
// 512 KiB a BF16 system of 6.7 MB takes 48 us an iteration for 25), 512 KiB in 8
// (in 256, 200 systems of 8 MB take 280 us for 271), and 128 rows of BF16 or 64 of
// FP32 (128 BF16 systems of 2000 x 4000 in cells of 64 rows 372 us, of 128 350; of
// 4000 x 1100 in 32 rows 242, in 128 220).
constexpr int64_t kMinItems = 8;
constexpr int64_t kMinItemKib = 32;
constexpr int32_t kMaxMinItems = 64;
struct BatchCut {
    int64_t rows_per_cell;
    int32_t cells;          // cells per group
};
inline int64_t cell_kib(int64_t elem_bytes, int64_t row_bytes) {
    return std::max({int64_t(256), 64 * elem_bytes, 256 / elem_bytes * row_bytes / 1024});
}
inline BatchCut plan_cut(int64_t m, int64_t ldA, int64_t elem_bytes, int32_t item_kib, int32_t min_items, int64_t unit,
                         int32_t max_cells) {
    const int64_t row_bytes = ldA * elem_bytes;
    const int64_t sys_kib = m * row_bytes / 1024, cap = std::max<int32_t>(1, item_kib);
    const int64_t least = min_items > 0 ? min_items : kMinItems;
    const int64_t kib = std::min(cap, std::max(kMinItemKib, sys_kib / least));
    BatchCut c{0, 1};
    if (min_items <= 0) c.cells = (int32_t)std::clamp<int64_t>(kib / cell_kib(elem_bytes, row_bytes), 1, max_cells);
    int64_t r = kib * 1024 / (row_bytes * c.cells);
    r = std::max(unit, (r + unit - 1) / unit * unit);
    c.rows_per_cell = std::min(r, (m + unit - 1) / unit * unit);
    return c;
}

// Cells of one work item: whole groups in a batch that has them for every CU,
// fewer cells in a smaller one, so that it has about kItemsPerWorkgroup items for
// each workgroup of the grid.  Cells that are written one by one spread a small
// batch over the device (seven BF16 systems of 78 MB in all: 210 us an iteration
// as 56 groups, 56 as 184 cells), but writing and reading back eight times the
// partials costs a larger one.  The line is at 7/4 groups of the largest size a CU
// (us an iteration by groups and by cells: FP32 1400 x 3000, 2.0 a CU 179 and 223,
// 4.0 351 and 423; FP64 700 x 3000, 1.5 160 and 154, 2.0 181 and 207; BF16
// 2000 x 4000, 1.5 179 and 172, 1.75 183 and 200; FP64 1000 x 10000, 1.25 516 and
// 448, 1.9 611 and 654).  A batch with larger groups is cut up anyway, and the
// systems between make better items as cells: only those are left whole whose
// groups are less than half the share of a workgroup (64 FP32 systems of 64 to
// 2048 columns: 125 us a sweep, 138 with the line of the even batches).
constexpr int64_t kItemsPerWorkgroup = 4;
inline int64_t plan_cells_per_item(const BatchCut &cut, int64_t row_bytes, int64_t batch_bytes, int64_t grid, int64_t cus,
                                   int64_t largest_group) {
    if (4 * batch_bytes >= 7 * cus * largest_group) return cut.cells;
    const int64_t want = batch_bytes / std::max<int64_t>(1, grid * kItemsPerWorkgroup);
    const int64_t cells = std::max<int64_t>(1, want / (cut.rows_per_cell * row_bytes));
    return 2 * cells > cut.cells ? cut.cells : cells;
}

// Workgroups of the batch sweep: `tuned` if positive, else every one that can be
// resident (per_cu a CU).  Fewer than two items for each of those: one workgroup
// per CU instead (a second one on some CUs slows the first, and the kernel waits
// for those; us an iteration, 16 FP64 systems of 17 MB 77 and 58, 16 FP32 of 7 MB
// 53 and 41, 64 FP64 of 2 MB 54 and 38; from two items on two are better, 128 FP64
// of 2 MB 60 and 64).  Not where min_items sets the cut: the autotuner, which sets
// it, compares cuts by sweeps without a translation, where one long item a system
// on one workgroup per CU looked best (512 FP32 systems of 256 x 2048: 165 us,
// two items 169) that lost with one (205, two items 195); grids it tries by itself.
inline int64_t plan_grid(int64_t tuned, int64_t per_cu, int64_t cus, int64_t items, int32_t min_items) {
    int64_t grid = tuned > 0 ? tuned : cus * per_cu;
    if (tuned <= 0 && min_items <= 0 && items < 2 * grid) grid = cus;
    return std::max<int64_t>(1, std::min(grid, std::max<int64_t>(1, items)));
}

// Row form of a system: rows of at most 64 16-byte vectors (C == 1) run four
// to a wavefront, 16 lanes each, with 1, 2 or 4 chunks per lane; longer rows
// (or with the short form switched off) one to a wavefront with C chunks.
inline void plan_row_form(int64_t ldA, int64_t vec_elems, int C, bool short_form, int32_t *rpw, int32_t *chunks) {
    *rpw = 1;
    *chunks = C;
    if (C != 1 || !short_form) return;
    *rpw = 4;
    const int64_t per = 16 * vec_elems;
    const int64_t k = (ldA + per - 1) / per;
    *chunks = k <= 1 ? 1 : k <= 2 ? 2 : 4;
}

}  // namespace modap_host
