// Host half of the library: the C ABI declared in include/modap.h.
//
// A context owns a device copy of the system (rows padded with zeros to a
// 16-byte multiple), its FP64 row norms, the approximation x, the last y, a
// one-shot translation slot, an optional drift schedule, the per-workgroup
// partials, the working vectors of the next sweep and a device control block.
// One iteration is two kernels on the context's stream: the fused sweep
// (which first settles the previous check: stop decision and step length)
// and the fixed-order reduction of y (which makes the previous step permanent
// in x and writes the next sweep's working vectors); a stage kernel settles
// the last check of a call.  The host never waits between iterations; solve()
// reads the control block once per batch of queued iterations.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <climits>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <iterator>
#include <string>
#include <thread>
#include <unordered_set>
#include <vector>

#include "aux_kernels.hpp"
#include "aux_launch.hpp"
#include "certify.hpp"
#include "host_common.hpp"
#include "trace.hpp"
#include "internal.hpp"
#include "modap.h"
#include "readback.hpp"
#include "resident.hpp"
#include "sweep_relay.hpp"
#include "sweep_split.hpp"
#include "modap_device.hpp"
#include "sweep_table.hpp"

using namespace modap;
using modap_host::Readback;

struct modap_ctx {
    int device = 0;
    hipStream_t stream = nullptr;
    int cu_count = 0;
    std::string err;

    // system
    bool loaded = false;
    int64_t m = 0, n = 0, ldA = 0;
    int dt = 0;
    size_t es = 0;
    void *A = nullptr;
    double *b = nullptr, *nu = nullptr, *x = nullptr, *y = nullptr, *vpend = nullptr;
    double *bref = nullptr;      // [m] right-hand side at zero translation: the data are bref + A wsum
    void *vectors = nullptr;     // the allocation of every vector of the system
    double *wsum = nullptr;      // [ldA] FP64 sum of the translations applied since the last rebase
    int *claim = nullptr;        // [m] row claims of a device-side replacement (zero between calls)
    double *V = nullptr;         // [T x ldA] drift schedule, in an allocation of V_cap doubles
    int64_t T = 0;
    size_t V_cap = 0;
    bool vpend_maybe = false;   // a translation may be pending on the device
    int64_t jn = 0;             // index of the next iteration; state of jn-1 is committed

    // kernel shape and scratch
    modap_tile tile{};
    bool tile_forced = false;
    const SweepKernel *kern_nov = nullptr, *kern_v = nullptr;
    // split-row two-phase form (tile kind 1)
    const SplitKernels *skern = nullptr;
    int ntiles = 0;
    int64_t rows_per_band = 0;
    int finish_blocks = 0;
    void *pdot = nullptr;
    size_t pdot_bytes = 0;
    double *wrow = nullptr;
    // one-read form of long rows (sweep_relay.hpp), used in place of the two phases
    bool relay_ok = false;
    bool relay_now = false;      // the last sweep queued took it
    int relay_tiles = 0, relay_bands = 0;
    int64_t relay_tile = 0, relay_rows = 0, relay_ldPart = 0;
    uint64_t *relay_words = nullptr;
    uint32_t relay_base = 0;     // number of the next launch's first row
    int64_t rows_per_block = 0;  // one-pass sweep: row mapping (see SweepArgs)
    int64_t block_stride = 0;
    int64_t step_stride = 0;
    int64_t ldPart = 0;
    void *part = nullptr;
    size_t part_bytes = 0;
    int64_t *h_part = nullptr;
    double *dmax_part = nullptr, *binf_part = nullptr;
    int part_grid = 0;
    double *ynp = nullptr;
    Totals *tot = nullptr;
    void *work = nullptr;        // [3 x ldA] accumulation type: x, v and y of the next sweep
    void *work_eval = nullptr;

    void *small = nullptr;       // the allocation of ctl, tot and checks
    Ctrl *ctl = nullptr;
    Readback rb;                 // results read back by the host (see readback.hpp)
    double *x_eval = nullptr, *y_eval = nullptr, *r_eval = nullptr;
    DataChecks *checks = nullptr;

    // staging for host-side update inputs
    void *stage = nullptr;
    size_t stage_bytes = 0;

    // resident iteration of small systems (resident.hpp): one launch of many
    // iterations on a few workgroups holding their rows in LDS
    bool res_ok = false;
    int res_grid = 0, res_rows = 0, res_ldR = 0;
    size_t res_lds = 0;
    uint64_t *res_words = nullptr;
    uint32_t res_base = 1;       // number of the next launch's first iteration

    // FP64 certificate (scratch allocated at the first certificate of a system)
    void *cert = nullptr;
    CertPlan cert_cut{};

    std::vector<hipEvent_t> events;
};

namespace {

using namespace modap_host;

const SweepKernel *kernels_for(int dt, int *count) {
    switch (dt) {
        case 0: return sweep_kernels_0(count);
        case 1: return sweep_kernels_1(count);
        default: return sweep_kernels_2(count);
    }
}

// The compiled kernel of a shape; depth 0 takes the shallowest one compiled.
const SweepKernel *find_kernel(int dt, int block, int lpr, int chunks, int rs, int depth, bool has_v) {
    int cnt = 0;
    const SweepKernel *t = kernels_for(dt, &cnt);
    const SweepKernel *hit = nullptr;
    for (int i = 0; i < cnt; ++i)
        if (t[i].block == block && t[i].lpr == lpr && t[i].chunks == chunks && t[i].rs == rs &&
            t[i].has_v == has_v && (depth == 0 ? (!hit || t[i].pd < hit->pd) : t[i].pd == depth))
            hit = &t[i];
    return hit;
}

int64_t coverage(int dt, int lpr, int chunks) { return (int64_t)lpr * vec_elems(dt) * chunks; }

const SplitKernels *split_for(int dt) {
    switch (dt) {
        case 0: return split_kernels_0();
        case 1: return split_kernels_1();
        default: return split_kernels_2();
    }
}

// Systems of at least this many bytes, cut into tiles of at least this many
// bytes a row, take the one-read form of long rows; below, the two phases are
// as fast or faster (us an iteration, one read and two phases, 4% of the rows
// violated: FP64 9000 x 1000 (72 MB) 44.8 and 41.9, 9000 x 2000 55.4 and 56.3,
// 9000 x 18000 224 and 265; BF16 17000 x 40000, whose tile rows have 11 KiB,
// 322 and 303, 30000 x 40000 (14.6 KiB) 422 and 436; with a third violated
// FP64 9000 x 18000 230 and 328, 14000 x 28000 497 and 691).
constexpr int64_t kRelayMinBytes = int64_t(128) << 20;
constexpr int64_t kRelayMinTileBytes = 14 * 1024;
constexpr int64_t kMaxBandRows = 4096;  // rows per band of the split-row form (its row list)

// Built-in choice of the fused sweep's shape, by storage type and padded row
// length: the first entry that holds a row.  The line between two entries is
// the coverage of the first (lanes x chunks x 16 bytes); why this shape at a
// length:
//  - rows of up to 256 bytes: 16 lanes a row, four rows to a wavefront;
//  - up to 8 KiB: a wavefront a row with all its chunks in registers.  No
//    barrier per row, and every wavefront keeps two or three rows in flight.
//    A row shared by 256 lanes pays a barrier and an exchange per row, which a
//    row of 8 KiB does not cover: BF16 4096 x 16384 took 46.8 us an iteration
//    at 256 lanes and 33.2 at 64, FP64 1000 x 4000 18.4 and 15.2, FP32
//    2000 x 6000 19.2 and 16.9; three or four rows of 16 lanes with four
//    chunks lose the same way (FP32 250 x 16384 14.4 and 13.0, BF16
//    500 x 32768 22.0 and 18.5);
//  - longer rows: the workgroup shares the row, in the fewest chunks that hold
//    it (BF16 12000 x 30000: 119.7 us with three chunks, 122.7 with four).
//    12-chunk wavefronts still beat 256 lanes on BF16 rows of 8 to 12 KiB
//    (6000 x 18000: 51.6 against 60.2).
//  - on systems of fewer rows than `few`, rows of a wavefront with six and more
//    chunks are spread over two or four wavefronts (the same vectors: 128 lanes
//    of 3 chunks for 64 of 6, 256 of 2 for 8, 256 of 3 for 12).  There a row's own
//    time counts, and below four rows a CU a band of four leaves CUs idle: BF16
//    4000 x 300 14.5 us an iteration with a wavefront a row and 11.0, 6000 x 2000
//    22.1 and 17.7, x 5000 27.3 and 25.1; FP64 1500 x 600 12.2 and 11.1, x 2500 15.4
//    and 15.6; FP32 2000 x 600 10.9 and 10.1, x 2000 12.5 and 13.0.
// Rows longer than the last entry take the split-row form.
struct ShapeFor {
    int32_t row;    // longest padded row
    int32_t block, lpr, chunks, rs, pd;
    int32_t few;    // systems of fewer rows spread the row over more lanes (0: none)
};
constexpr ShapeFor kShapesF64[] = {
    {32, 256, 16, 1, 1, 2},      {64, 256, 16, 2, 1, 2},      {128, 256, 16, 4, 1, 2},   {256, 256, 64, 2, 2, 2},
    {384, 256, 64, 3, 2, 2},     {512, 256, 64, 4, 1, 2},     {768, 256, 64, 6, 1, 3, 1000},
    {1024, 256, 64, 8, 1, 2, 1000}, {1536, 256, 64, 12, 1, 2, 2000},
    {2048, 256, 256, 4, 1, 4},   {3072, 256, 256, 6, 1, 2},   {4096, 256, 256, 8, 1, 2}, {6144, 512, 512, 6, 1, 2},
    {8192, 512, 512, 8, 1, 2}};
constexpr ShapeFor kShapesF32[] = {
    {64, 256, 16, 1, 1, 2},      {128, 256, 16, 2, 1, 2},     {256, 512, 64, 1, 1, 4},   {512, 512, 64, 2, 2, 2},
    {768, 256, 64, 3, 1, 3},     {1024, 256, 64, 4, 1, 2},    {1536, 256, 64, 6, 1, 3, 1500},
    {2048, 256, 64, 8, 1, 2, 1500},
    {4096, 512, 256, 4, 1, 2},   {6144, 256, 256, 6, 1, 2},   {8192, 256, 256, 8, 1, 2}, {12288, 512, 512, 6, 1, 2},
    {16384, 512, 512, 8, 1, 2}};
constexpr ShapeFor kShapesBF16[] = {
    {128, 256, 16, 1, 1, 2},     {256, 256, 16, 2, 1, 2},     {512, 256, 64, 1, 2, 2},   {1024, 256, 64, 2, 1, 2},
    {1536, 256, 64, 3, 1, 3},    {2048, 256, 64, 4, 1, 2},    {3072, 256, 64, 6, 1, 2, 3500},
    {4096, 256, 64, 8, 1, 3, 3500}, {6144, 256, 64, 12, 1, 2, 5000},
    {8192, 512, 512, 2, 2, 2},   {12288, 512, 512, 3, 1, 2},  {16384, 512, 512, 4, 1, 2}};

// Two more exceptions by the number of rows.  FP64 rows of 65 to 128 elements: four
// rows to a wavefront leave compute units idle on short systems (120 x 480:
// 9.8 us against 8.4 with a wavefront a row, 120 x 4096 12.3 and 11.5, but
// 120 x 16384 14.9 and 16.1).  And 16-lane rows of long systems take two
// workgroups per CU, whose partials are short (BF16 100 x 131072: 21.0 us
// against 25.2; FP32 120 x 65536 17.2 and 18.3, 120 x 16384 13.6 and 12.2).
constexpr int64_t kFewRowsF64 = 8192;
constexpr int64_t kManyRows = 65536;

void choose_shape(int dt, int64_t ldA, int64_t m, int cu_count, modap_tile *out) {
    const ShapeFor *t = dt == 0 ? kShapesF64 : dt == 1 ? kShapesF32 : kShapesBF16;
    const ShapeFor *end = dt == 0 ? std::end(kShapesF64) : dt == 1 ? std::end(kShapesF32) : std::end(kShapesBF16);
    while (t != end && t->row < ldA) ++t;
    *out = modap_tile{};
    if (t == end) {
        const SplitKernels *sk = split_for(dt);
        out->kind = 1;
        out->block = sk->block;
        out->lanes_per_row = sk->block;
        out->chunks = sk->chunks;
        out->rows_per_step = 1;
        return;
    }
    out->block = t->block;
    out->lanes_per_row = t->lpr;
    out->chunks = t->chunks;
    out->rows_per_step = t->rs;
    out->depth = t->pd;
    if (m < t->few) {
        out->block = 256;
        out->lanes_per_row = t->chunks == 6 ? 128 : 256;
        out->chunks = t->chunks * t->lpr / out->lanes_per_row;
        out->rows_per_step = 1;
        out->depth = 2;
    } else if (dt == 0 && t->row == 128 && m < kFewRowsF64) {
        out->lanes_per_row = 64;
        out->chunks = 1;
    } else if (t->lpr < 64 && m >= kManyRows) {
        out->grid = 2 * cu_count;
    }
}

modap_status ensure_scalar_parts(modap_ctx *c, int count) {
    if (count <= c->part_grid) return MODAP_OK;
    free_dev(c->h_part);
    free_dev(c->dmax_part);
    free_dev(c->binf_part);
    c->part_grid = 0;
    HIP_TRY(c, hipMalloc(&c->h_part, sizeof(int64_t) * count));
    HIP_TRY(c, hipMalloc(&c->dmax_part, sizeof(double) * count));
    HIP_TRY(c, hipMalloc(&c->binf_part, sizeof(double) * count));
    c->part_grid = count;
    return MODAP_OK;
}

modap_status ensure_part(modap_ctx *c, size_t need) {
    HIP_TRY(c, grow_dev(c->part, c->part_bytes, need, 1));
    return MODAP_OK;
}

// Split-row form: column tiles of 256*VEC*C columns, row bands of at most
// kMaxBandRows rows; grid = number of row bands (0: about two workgroups per
// compute unit over bands x tiles).
modap_status configure_split(modap_ctx *c, modap_tile t) {
    const SplitKernels *sk = split_for(c->dt);
    if (t.block != sk->block || t.lanes_per_row != sk->block || t.chunks != sk->chunks)
        return fail(c, MODAP_E_INVAL, "no compiled split-row kernel of that shape for this storage type");
    const int64_t tw = (int64_t)sk->block * vec_elems(c->dt) * sk->chunks;
    const int ntiles = (int)((c->ldA + tw - 1) / tw);
    int64_t bands = t.grid > 0 ? t.grid : std::max<int64_t>(1, (2 * c->cu_count + ntiles - 1) / ntiles);
    int64_t rpb = (c->m + bands - 1) / bands;
    rpb = std::min(rpb, kMaxBandRows);
    bands = (c->m + rpb - 1) / rpb;
    const size_t acc = acc_size(c->dt);
    modap_status st;
    if ((st = ensure_part(c, (size_t)bands * (size_t)ntiles * (size_t)tw * acc))) return st;
    const size_t pd = 2 * (size_t)ntiles * (size_t)c->m * acc;
    HIP_TRY(c, grow_dev(c->pdot, c->pdot_bytes, pd, 1));
    if (!c->wrow) HIP_TRY(c, hipMalloc(&c->wrow, sizeof(double) * (size_t)c->m));
    c->finish_blocks = (int)((c->m + 255) / 256);
    if ((st = ensure_scalar_parts(c, c->finish_blocks))) return st;
    c->skern = sk;
    c->ntiles = ntiles;
    c->rows_per_band = rpb;
    c->ldPart = (int64_t)ntiles * tw;
    t.grid = (int)bands;
    t.rows_per_step = 1;
    t.depth = 0;
    t.interleave = 0;
    c->tile = t;
    c->kern_v = c->kern_nov = nullptr;
    return MODAP_OK;
}

// Resolve the tile into kernels, grid and scratch.
modap_status configure(modap_ctx *c, const modap_tile &want) {
    modap_tile t = want;
    if (t.kind == 1) return configure_split(c, t);
    if (t.kind != 0) return fail(c, MODAP_E_INVAL, "tile kind must be 0 (one pass) or 1 (split rows)");
    if (t.rows_per_step <= 0) t.rows_per_step = 1;
    if (t.depth < 0) return fail(c, MODAP_E_INVAL, "tile depth must be >= 0");
    const SweepKernel *kv = find_kernel(c->dt, t.block, t.lanes_per_row, t.chunks, t.rows_per_step, t.depth, true);
    if (!kv) return fail(c, MODAP_E_INVAL, "no compiled sweep kernel of that shape for this storage type");
    t.depth = kv->pd;
    const SweepKernel *kn = find_kernel(c->dt, t.block, t.lanes_per_row, t.chunks, t.rows_per_step, t.depth, false);
    if (!kn) return fail(c, MODAP_E_INVAL, "no compiled sweep kernel of that shape for this storage type");
    const int64_t cov = coverage(c->dt, t.lanes_per_row, t.chunks);
    if (cov < c->ldA) return fail(c, MODAP_E_INVAL, "sweep shape does not cover a row");
    const int per_step = (t.block / t.lanes_per_row) * t.rows_per_step;
    // By default one workgroup per CU: with every row group keeping depth-1
    // steps of rows in flight, a second workgroup per CU adds no bandwidth
    // but doubles the partial y written at the end of the sweep.
    int grid = t.grid > 0 ? t.grid : c->cu_count;
    if (t.interleave != 0 && t.interleave != 1) return fail(c, MODAP_E_INVAL, "tile interleave must be 0 or 1");
    int64_t rpb, block_stride, step_stride;
    if (t.interleave) {
        // workgroup b takes row blocks b, b + grid, b + 2*grid, ... of per_step rows
        grid = (int)std::min<int64_t>(grid, (c->m + per_step - 1) / per_step);
        rpb = c->m;
        block_stride = per_step;
        step_stride = (int64_t)grid * per_step;
    } else {
        rpb = (c->m + grid - 1) / grid;
        rpb = ((rpb + per_step - 1) / per_step) * per_step;
        grid = (int)((c->m + rpb - 1) / rpb);
        block_stride = rpb;
        step_stride = per_step;
    }
    const size_t acc = acc_size(c->dt);
    modap_status st;
    if ((st = ensure_part(c, (size_t)grid * (size_t)cov * acc))) return st;
    if ((st = ensure_scalar_parts(c, grid))) return st;
    c->skern = nullptr;
    c->kern_v = kv;
    c->kern_nov = kn;
    c->rows_per_block = rpb;
    c->block_stride = block_stride;
    c->step_stride = step_stride;
    c->ldPart = cov;
    t.grid = grid;
    c->tile = t;
    return MODAP_OK;
}

modap_status check_ctx(modap_ctx *c, bool need_system) {
    if (!c) return MODAP_E_INVAL;
    if (need_system && !c->loaded) return fail(c, MODAP_E_STATE, "no system loaded (call modap_set_system first)");
    return MODAP_OK;
}

modap_status check_params(modap_ctx *c, const modap_params *p) {
    const char *msg = nullptr;
    const modap_status st = modap_host::check_params(p, &msg);
    return st ? fail(c, st, msg) : MODAP_OK;
}


modap_status ensure_stage(modap_ctx *c, size_t bytes) {
    if (bytes <= c->stage_bytes) return MODAP_OK;
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    HIP_TRY(c, grow_dev(c->stage, c->stage_bytes, bytes, 1));
    return MODAP_OK;
}

// Copy caller data (host or device) to a device pointer, stream-ordered.
modap_status to_device(modap_ctx *c, void *dst, const void *src, size_t bytes, int on_dev) {
    if (bytes == 0) return MODAP_OK;
    HIP_TRY(c, hipMemcpyAsync(dst, src, bytes, on_dev ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice, c->stream));
    return MODAP_OK;
}

modap_status from_device(modap_ctx *c, void *dst, const void *src, size_t bytes, int on_dev) {
    if (bytes == 0) return MODAP_OK;
    HIP_TRY(c, hipMemcpyAsync(dst, src, bytes, on_dev ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, c->stream));
    return MODAP_OK;
}

double sweep_bytes(const modap_ctx *c, bool with_v) {
    return (double)c->m * (double)c->n * (double)c->es + 16.0 * (double)c->m + (with_v ? 8.0 * (double)c->m : 0.0);
}

bool translation_possible(const modap_ctx *c) { return c->vpend_maybe || (c->V && c->T > 0); }

int reduce_grid(const modap_ctx *c) { return (int)((c->n + 63) / 64); }

size_t relay_word_bytes(const modap_ctx *c) {
    return sizeof(uint64_t) * (size_t)c->relay_bands * (size_t)kRelayRing * (size_t)relay_row_words(c->relay_tiles);
}

// Longest wait of a resident launch for its other workgroups, and of a long-row
// sweep for a peer's dot product, in ticks of the 100 MHz constant clock.
constexpr int64_t kTimeoutTicks = 100000000;   // one second
int64_t timeout_ticks() {
    const char *e = std::getenv("MODAP_RESIDENT_TIMEOUT_TICKS");
    return e ? std::atoll(e) : kTimeoutTicks;
}

int last_slot(const modap_ctx *c) { return (int)((c->jn - 1) & 1); }

Decide decide_params(const modap_params *p, int track) {
    Decide d{};
    d.lambda = p->lambda;
    d.eps = p->eps;
    d.eps_relative = p->eps_relative;
    d.rule = p->step;
    d.track = track;
    return d;
}

SweepArgs sweep_args(modap_ctx *c) {
    SweepArgs a{};
    a.A = c->A;
    a.ldA = c->ldA;
    a.m = c->m;
    a.n = c->n;
    a.b_in = c->b;
    a.nu = c->nu;
    a.work = c->work;
    a.pd.ctl = c->ctl;
    a.pd.j = c->jn;
    a.pd.tot = c->tot;
    a.pd.ynp = c->ynp;
    a.pd.R = reduce_grid(c);
    a.pd.decide = 0;
    a.part = c->part;
    a.ldPart = c->ldPart;
    a.h_part = c->h_part;
    a.dmax_part = c->dmax_part;
    a.binf_part = c->binf_part;
    a.rows_per_block = c->rows_per_block;
    a.block_stride = c->block_stride;
    a.step_stride = c->step_stride;
    return a;
}

// What is queued may be run again later (a stream that cannot be asked counts as one under capture).
bool under_capture(const modap_ctx *c) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(c->stream, &cap) != hipSuccess) {
        (void)hipGetLastError();
        return true;
    }
    return cap != hipStreamCaptureStatusNone;
}

// The one-read form of long rows serves the built-in choice of the split-row
// form.  Its launch is cooperative and its rows are numbered by the host, so a
// stream under capture takes the two phases.
bool use_relay(const modap_ctx *c) { return c->relay_ok && !c->tile_forced && c->skern && !under_capture(c); }

// Launch the sweep of the configured form (events: start/end of its kernels).
modap_status launch_sweep(modap_ctx *c, const SweepArgs &a, bool hv, hipEvent_t e0, hipEvent_t e1) {
    c->relay_now = use_relay(c);
    if (!c->skern) {
        HIP_TRY(c, (hv ? c->kern_v : c->kern_nov)->launch(a, c->tile.grid, c->stream, e0, e1));
        return MODAP_OK;
    }
    SplitArgs s{};
    s.A = a.A;
    s.ldA = a.ldA;
    s.m = a.m;
    s.n = a.n;
    s.b_in = a.b_in;
    s.b_out = a.b_out;
    s.nu = a.nu;
    s.work = a.work;
    s.pd = a.pd;
    s.check_status = a.check_status;
    s.ntiles = c->ntiles;
    s.rows_per_band = c->rows_per_band;
    s.pdot = c->pdot;
    s.w = c->wrow;
    s.r_out = a.r_out;
    s.part = c->part;
    s.ldPart = c->ldPart;
    s.h_part = c->h_part;
    s.dmax_part = c->dmax_part;
    s.binf_part = c->binf_part;
    if (e0) HIP_TRY(c, hipEventRecord(e0, c->stream));
    if (c->relay_now) {
        // numbers of rows are used once; long before they come round the words start afresh
        if (c->relay_base > 0xf0000000u) {
            HIP_TRY(c, hipMemsetAsync(c->relay_words, 0, relay_word_bytes(c), c->stream));
            c->relay_base = 1;
        }
        RelayArgs r{};
        s.ntiles = c->relay_tiles;
        s.rows_per_band = c->relay_rows;
        s.ldPart = c->relay_ldPart;
        r.s = s;
        r.tile = c->relay_tile;
        r.words = c->relay_words;
        r.base = c->relay_base;
        r.timeout_ticks = timeout_ticks();
        HIP_TRY(c, c->skern->relay(r, c->relay_bands * c->relay_tiles, hv, c->stream));
        c->relay_base += (uint32_t)c->relay_rows;
        if (e1) HIP_TRY(c, hipEventRecord(e1, c->stream));
        return MODAP_OK;
    }
    HIP_TRY(c, c->skern->dot(s, c->tile.grid, c->ntiles, hv, c->stream));
    HIP_TRY(c, c->skern->finish(s, c->finish_blocks, hv, c->stream));
    HIP_TRY(c, c->skern->axpy(s, c->tile.grid, c->ntiles, c->stream));
    if (e1) HIP_TRY(c, hipEventRecord(e1, c->stream));
    return MODAP_OK;
}

ReduceArgs reduce_args(modap_ctx *c) {
    ReduceArgs r{};
    r.part = c->part;
    r.ldPart = c->relay_now ? c->relay_ldPart : c->ldPart;
    r.G = c->relay_now ? c->relay_bands : c->tile.grid;
    r.Gs = c->relay_now ? c->relay_bands : c->skern ? c->finish_blocks : c->tile.grid;
    r.acc_f64 = c->dt == 0;
    r.n = c->n;
    r.ldA = c->ldA;
    r.x = c->x;
    r.V = c->V;
    r.ldV = c->ldA;
    r.h_part = c->h_part;
    r.dmax_part = c->dmax_part;
    r.binf_part = c->binf_part;
    r.tot = c->tot;
    r.ynp = c->ynp;
    r.vpend = c->vpend;
    return r;
}

modap_status launch_reduce(modap_ctx *c, const ReduceArgs &r, hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr) {
    if (e0 || e1) {
        ReduceArgs copy = r;
        void *args[] = {&copy};
        const void *f = r.acc_f64 ? reinterpret_cast<const void *>(&reduce_y<double>)
                                  : reinterpret_cast<const void *>(&reduce_y<float>);
        HIP_TRY(c, hipExtLaunchKernel(f, dim3(reduce_grid(c)), dim3(kReduceThreads), args, 0, c->stream, e0, e1, 0));
        return MODAP_OK;
    }
    if (r.acc_f64)
        hipLaunchKernelGGL(reduce_y<double>, dim3(reduce_grid(c)), dim3(kReduceThreads), 0, c->stream, r);
    else
        hipLaunchKernelGGL(reduce_y<float>, dim3(reduce_grid(c)), dim3(kReduceThreads), 0, c->stream, r);
    LAUNCH_TRY(c, "reduce_y launch");
    return MODAP_OK;
}

hipEvent_t event_at(modap_ctx *c, size_t i) {
    while (c->events.size() <= i) {
        hipEvent_t e = nullptr;
        if (hipEventCreate(&e) != hipSuccess) return nullptr;
        c->events.push_back(e);
    }
    return c->events[i];
}

// Create the events of `iters` queued iterations of which every `every`-th is
// profiled, before any is queued: creating one while the device runs ahead
// of the host would leave the device idle.
modap_status reserve_events(modap_ctx *c, int64_t iters, int64_t every) {
    if (every <= 0 || iters <= 0) return MODAP_OK;
    const int64_t need = 4 * ((iters + every - 1) / every);
    if (!event_at(c, (size_t)need - 1)) return fail(c, MODAP_E_DEVICE, "hipEventCreate failed");
    return MODAP_OK;
}

// Profiling: events 4i..4i+3 of iteration i mark the sweep's start and end
// and the reduction's start and end, recorded by the kernel dispatches
// themselves.
bool profile_events(modap_ctx *c, size_t first, hipEvent_t (&e)[4]) {
    for (int k = 0; k < 4; ++k) {
        e[k] = event_at(c, first + k);
        if (!e[k]) return false;
    }
    return true;
}

StageArgs stage_args(modap_ctx *c, const modap_params *p, int track, int64_t j) {
    StageArgs g{};
    g.ctl = c->ctl;
    g.j = j;
    g.tot = c->tot;
    g.ynp = c->ynp;
    g.R = reduce_grid(c);
    if (p) g.dp = decide_params(p, track);
    g.x = c->x;
    g.y = c->y;
    g.vpend = c->vpend;
    g.V = c->V;
    g.ldV = c->ldA;
    g.n = c->n;
    g.ldA = c->ldA;
    g.work = c->work;
    return g;
}

int stage_grid(const modap_ctx *c) { return (int)std::min<int64_t>(1024, (c->n + 255) / 256); }

// Working vectors of the next sweep from the committed state (call start).
modap_status enqueue_prime(modap_ctx *c, void *work, const double *x) {
    StageArgs g = stage_args(c, nullptr, 0, c->jn);
    g.x = const_cast<double *>(x);
    g.work = work;
    if (c->dt == 0)
        hipLaunchKernelGGL(prime_work<double>, dim3(stage_grid(c)), dim3(256), 0, c->stream, g);
    else
        hipLaunchKernelGGL(prime_work<float>, dim3(stage_grid(c)), dim3(256), 0, c->stream, g);
    LAUNCH_TRY(c, "prime_work launch");
    return MODAP_OK;
}

// Queue iteration i of a call: the sweep (which first settles the previous
// check, except in the first iteration of a call) at the current x on the
// current data, then the reduction of y (which makes the previous step
// permanent in x and writes the next sweep's working vectors).
modap_status enqueue_iteration(modap_ctx *c, const modap_params *p, int track, int64_t i, uint64_t *progress,
                               size_t *ev_used, double *bytes) {
    const bool hv = translation_possible(c);
    const int64_t j = c->jn;
    hipEvent_t ev[4] = {nullptr, nullptr, nullptr, nullptr};
    if (p->profile > 0 && i % p->profile == 0) {
        if (!profile_events(c, *ev_used, ev)) return fail(c, MODAP_E_DEVICE, "hipEventCreate failed");
        *ev_used += 4;
    }
    SweepArgs a = sweep_args(c);
    a.b_out = c->b;
    a.pd.j = j;
    a.pd.decide = i > 0;   // the first sweep of a call runs under the committed state
    a.pd.dp = decide_params(p, track);
    a.pd.progress = progress;
    a.check_status = 1;
    modap_status st;
    if ((st = launch_sweep(c, a, hv, ev[0], ev[1]))) return st;
    ReduceArgs r = reduce_args(c);
    r.y = c->y;
    r.ctl = c->ctl;
    r.j = j;
    r.iterate = 1;
    r.apply_step = i > 0;
    r.work = c->work;
    r.wsum = hv ? c->wsum : nullptr;   // no translation: nothing to add to the sum
    r.has_v = hv;
    if ((st = launch_reduce(c, r, ev[2], ev[3]))) return st;
    c->jn = j + 1;
    *bytes += sweep_bytes(c, hv);
    return MODAP_OK;
}

// End of a call that queued iterations: settle the last check (decision,
// step) with the stage kernel, so the committed state is in slot (jn-1)&1.
modap_status enqueue_settle(modap_ctx *c, const modap_params *p, int track) {
    StageArgs g = stage_args(c, p, track, c->jn - 1);
    if (c->dt == 0)
        hipLaunchKernelGGL(stage_iter<double>, dim3(stage_grid(c)), dim3(256), 0, c->stream, (const StageArgs)g);
    else
        hipLaunchKernelGGL(stage_iter<float>, dim3(stage_grid(c)), dim3(256), 0, c->stream, (const StageArgs)g);
    LAUNCH_TRY(c, "stage_iter launch");
    return MODAP_OK;
}

modap_status fault_status(modap_ctx *c) {
    return fail(c, MODAP_E_DEVICE,
                "a launch gave up waiting for its other workgroups; the context's data are void until set_system");
}

// Wait for everything queued and read the committed state (and, for a query,
// up to two vectors of doubles to host memory).
modap_status read_back(modap_ctx *c, State *out, const double *src0 = nullptr, double *dst0 = nullptr, int64_t n0 = 0,
                       const double *src1 = nullptr, double *dst1 = nullptr, int64_t n1 = 0) {
    PublishArgs p{};
    p.st = &c->ctl->st[last_slot(c)];
    p.fault = &c->ctl->fault;
    const double *src[2] = {src0, src1};
    double *dst[2] = {dst0, dst1};
    const int64_t cnt[2] = {n0, n1};
    const bool staged = n0 + n1 <= Readback::kMaxStaged;
    if (staged) {
        HIP_TRY(c, c->rb.reserve(n0 + n1));
        p.src[0] = src0;
        p.src[1] = src1;
        p.dst[0] = c->rb.buf_dev;
        p.dst[1] = c->rb.buf_dev + n0;
        p.count[0] = n0;
        p.count[1] = n1;
    } else {
        for (int k = 0; k < 2; ++k)
            if (cnt[k]) HIP_TRY(c, hipMemcpyAsync(dst[k], src[k], sizeof(double) * (size_t)cnt[k], hipMemcpyDeviceToHost, c->stream));
    }
    HIP_TRY(c, c->rb.run(p, c->stream));
    if (staged) {
        if (n0) std::memcpy(dst0, c->rb.buf, sizeof(double) * (size_t)n0);
        if (n1) std::memcpy(dst1, c->rb.buf + n0, sizeof(double) * (size_t)n1);
    }
    *out = c->rb.view->st;
    return c->rb.view->fault ? fault_status(c) : MODAP_OK;
}

void fill_stats(modap_stats *o, const State &k) {
    o->iters = k.steps;
    o->sweeps = k.sweeps;
    o->converged = k.feasible;
    o->state = k.status;
    o->max_viol = k.dmax;
    o->h = k.h;
    o->y_norm = k.ynorm;
    o->b_inf = k.binf;
    o->eps_abs = k.eps_abs;
    o->certified = k.certified;
    o->b_drift = k.bdrift;
}

modap_status profile_totals(modap_ctx *c, size_t ev_used, modap_stats *o) {
    double sw = 0.0, rd = 0.0;
    int64_t cnt = 0;
    for (size_t i = 0; i + 3 < ev_used; i += 4) {
        float a = 0.f, b = 0.f;
        HIP_TRY(c, hipEventElapsedTime(&a, c->events[i], c->events[i + 1]));
        HIP_TRY(c, hipEventElapsedTime(&b, c->events[i + 2], c->events[i + 3]));
        sw += a;
        rd += b;
        ++cnt;
    }
    o->sweep_ms = sw;
    o->reduce_ms = rd;
    o->profiled = cnt;
    return MODAP_OK;
}

modap_status status_of(modap_ctx *c, const State &k, bool solve) {
    switch (k.status) {
        case ST_RUNNING:
        case ST_CONVERGED: return MODAP_OK;
        case ST_LIMIT: return solve ? fail(c, MODAP_E_NOT_CONVERGED, "step limit reached before eps-feasibility") : MODAP_OK;
        case ST_NO_DIRECTION: return fail(c, MODAP_E_INFEASIBLE, "a row is violated but y = 0: no step direction");
        case ST_NUMERIC: return fail(c, MODAP_E_NUMERIC, "NaN or infinity in the iteration");
        case ST_BAD_ROW: return fail(c, MODAP_E_ZERO_ROW, "a replaced row is zero, not finite, out of range or repeated");
        case ST_UNCERTIFIED:
            return fail(c, MODAP_E_NOT_CONVERGED, "the FP64 certificate cannot confirm the stop: eps_abs lies below "
                                                  "its rounding bound");
        default: return fail(c, MODAP_E_DEVICE, "unknown device state");
    }
}

void release_resident(modap_ctx *c) {
    free_dev(c->res_words);
    c->res_ok = false;
}

void release_system(modap_ctx *c) {
    free_dev(c->cert);
    free_dev(c->relay_words);
    c->relay_ok = false;
    release_resident(c);
    free_dev(c->A);
    free_dev(c->vectors);
    free_dev(c->wrow);
    free_dev(c->V);
    c->V_cap = 0;
    c->T = 0;
    c->loaded = false;
}

modap_status launch_scatter(modap_ctx *c, int64_t k, const int64_t *rows, const void *new_rows, const double *nb) {
    HIP_TRY(c, aux_scatter_rows(c->dt, c->A, c->ldA, c->m, c->n, k, rows, new_rows, nb, c->b, c->bref, c->nu,
                                c->ctl, last_slot(c), c->vpend, c->V, c->ldA, c->wsum, c->stream));
    return MODAP_OK;
}

// Resident iteration (resident.hpp): systems whose rows hold at most 512
// elements and whose A, with rows padded to a multiple of 64 elements, fits
// in the LDS of at most kResidentMaxGrid workgroups at kResidentBand bytes
// each.  The grid is the larger of that minimum and one workgroup per
// kResidentRows rows (fewer rows per workgroup shorten the sweep; more
// workgroups lengthen the exchange).
constexpr int64_t kResidentBand = 96 * 1024;
constexpr int64_t kResidentRows = 32;

modap_status plan_resident(modap_ctx *c) {
    release_resident(c);
    const int64_t ldR = (c->n + 63) / 64 * 64;
    if (ldR > kResidentMaxCols) return MODAP_OK;
    const int64_t row_bytes = ldR * (int64_t)c->es;
    const int64_t gmin = (c->m * row_bytes + kResidentBand - 1) / kResidentBand;
    if (gmin > kResidentMaxGrid) return MODAP_OK;
    int64_t rows_target = kResidentRows;
    if (const char *e = std::getenv("MODAP_RESIDENT_ROWS")) rows_target = std::max<int64_t>(4, std::atoll(e));
    int64_t grid = std::min<int64_t>(kResidentMaxGrid, std::max(gmin, (c->m + rows_target - 1) / rows_target));
    const int64_t rows = (c->m + grid - 1) / grid;
    grid = (c->m + rows - 1) / rows;
    const size_t lds = resident_lds_bytes(c->dt, (int)rows, (int)ldR);
    int max_lds = 0;
    if (hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, c->device) != hipSuccess ||
        lds + kResidentStaticLds > (size_t)max_lds)
        return MODAP_OK;
    const size_t words = (size_t)resident_all_words(c->dt, (int)ldR, kResidentMaxGrid);
    HIP_TRY(c, hipMalloc(&c->res_words, sizeof(uint64_t) * words));
    HIP_TRY(c, hipMemsetAsync(c->res_words, 0, sizeof(uint64_t) * words, c->stream));
    c->res_base = 1;
    c->res_grid = (int)grid;
    c->res_rows = (int)rows;
    c->res_ldR = (int)ldR;
    c->res_lds = lds;
    c->res_ok = true;
    return MODAP_OK;
}

// The one-read form of long rows (sweep_relay.hpp): one workgroup per CU, the
// columns in tiles of equal width (a multiple of 128 bytes), as many bands of
// rows as CUs remain per tile.
modap_status plan_relay(modap_ctx *c) {
    c->relay_ok = false;
    modap_tile t{};
    choose_shape(c->dt, c->ldA, c->m, c->cu_count, &t);
    if (t.kind != 1 || c->m * c->ldA * (int64_t)c->es < kRelayMinBytes) return MODAP_OK;
    const int64_t most = relay_tile(c->dt), line = 128 / (int64_t)c->es;
    const int64_t tiles = (c->ldA + most - 1) / most;
    if (tiles > kRelayMaxTiles || tiles > c->cu_count || c->ldA / tiles * (int64_t)c->es < kRelayMinTileBytes)
        return MODAP_OK;
    int per_cu = 0;
    const void *f = split_for(c->dt)->relay_fn;
    if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)relay_hold(c->dt)) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, f, kRelayThreads + 128, relay_hold(c->dt)) != hipSuccess ||
        per_cu < 1) {
        (void)hipGetLastError();
        return MODAP_OK;
    }
    int64_t bands = c->cu_count / tiles;
    const int64_t rows = (c->m + bands - 1) / bands;
    bands = (c->m + rows - 1) / rows;
    c->relay_tiles = (int)tiles;
    c->relay_tile = std::min(most, ((c->ldA + tiles - 1) / tiles + line - 1) / line * line);
    c->relay_rows = rows;
    c->relay_bands = (int)bands;
    c->relay_ldPart = (c->ldA + 63) / 64 * 64;
    modap_status st;
    if ((st = ensure_part(c, (size_t)bands * (size_t)c->relay_ldPart * acc_size(c->dt)))) return st;
    if ((st = ensure_scalar_parts(c, (int)bands))) return st;
    HIP_TRY(c, hipMalloc(&c->relay_words, relay_word_bytes(c)));
    HIP_TRY(c, hipMemsetAsync(c->relay_words, 0, relay_word_bytes(c), c->stream));
    c->relay_base = 1;
    c->relay_ok = true;
    return MODAP_OK;
}

// The resident path runs unless the caller forced a tile of the two-kernel
// sweep, asked for per-iteration kernel timings, or set MODAP_RESIDENT=0.
bool use_resident(const modap_ctx *c, const modap_params *p) {
    if (!c->res_ok || c->tile_forced || p->profile > 0) return false;
    const char *e = std::getenv("MODAP_RESIDENT");
    return !(e && e[0] == '0');
}

// Queue K resident iterations from the committed state (the launch settles
// every check it makes, so no stage kernel follows).
modap_status launch_resident(modap_ctx *c, const modap_params *p, int track, int64_t K, uint64_t *progress,
                             double *bytes) {
    const bool hv = translation_possible(c);
    ResidentArgs r{};
    r.A = c->A;
    r.ldA = c->ldA;
    r.m = c->m;
    r.n = c->n;
    r.ldR = c->res_ldR;
    r.rows = c->res_rows;
    r.b = c->b;
    r.nu = c->nu;
    r.x = c->x;
    r.y = c->y;
    r.wsum = c->wsum;
    r.vpend = c->vpend;
    r.V = c->V;
    r.ldV = c->ldA;
    r.work = c->work;
    r.ctl = c->ctl;
    r.j0 = c->jn;
    r.K = K;
    r.dp = decide_params(p, track);
    // Words are told apart by the numbers of their iterations, which the host
    // gives out once.  A captured launch gives the same ones again each time it is
    // replayed, and 32 bits of them come round: such a launch starts with clear
    // words (cleared by a kernel: memory-set nodes have given wrong results in replays).
    const bool comes_round = (uint64_t)c->res_base + (uint64_t)K > UINT32_MAX;
    if (comes_round) c->res_base = 1;
    if (comes_round || under_capture(c)) {
        hipLaunchKernelGGL(clear_words, dim3(64), dim3(256), 0, c->stream, c->res_words,
                           resident_all_words(c->dt, c->res_ldR, kResidentMaxGrid));
        LAUNCH_TRY(c, "clear_words launch");
    }
    r.words = c->res_words;
    r.base = c->res_base;
    r.progress = progress;
    r.timeout_ticks = timeout_ticks();
    HIP_TRY(c, aux_resident_launch(c->dt, r, c->res_grid, c->res_lds, c->stream));
    c->res_base += (uint32_t)K;
    c->jn += K;
    *bytes += (double)K * sweep_bytes(c, hv);
    return MODAP_OK;
}

// Iterations a solve keeps queued beyond the last decision the host has seen:
// enough to cover the decision's way to the host and the next launch's to the
// device (about 10 us; an iteration takes about 10 us plus its bytes at 6
// TB/s), few enough that a stop leaves little queued in vain.  Queued in
// doubling chunks instead, a solve of 16 steps on a 128 MB system launched 126
// iterations and took 2.4 ms.
int64_t solve_ahead(const modap_ctx *c) {
    const double us = 10.0 + sweep_bytes(c, true) / 6e6;
    return us > 100.0 ? 2 : 4;
}

// One turn of a host loop that polls: a pause, and now and then a look at the
// stream for an error, and a yield once the wait has become long.
modap_status poll_pause(modap_ctx *c, uint32_t turn) {
    _mm_pause();
    if ((turn & 0x3fff) == 0) {
        const hipError_t e = hipStreamQuery(c->stream);
        if (e != hipSuccess && e != hipErrorNotReady) return hip_fail(c, e, "hipStreamQuery");
        (void)hipGetLastError();
        std::this_thread::yield();
    }
    return MODAP_OK;
}

// Queue the FP64 certificate of the committed state (a no-op on the device
// unless that state is an uncertified stop).
modap_status enqueue_certify(modap_ctx *c, const modap_params *p) {
    if (!c->cert) {
        // eight workgroups per CU keep the pass over A at the HBM rate
        c->cert_cut = cert_plan(c->dt, c->m, c->n, c->ldA, 8 * (int64_t)c->cu_count);
        HIP_TRY(c, hipMalloc(&c->cert, c->cert_cut.bytes));
    }
    CertArgs v{};
    v.A = c->A;
    v.ldA = c->ldA;
    v.m = c->m;
    v.n = c->n;
    v.b = c->b;
    v.bref = c->bref;
    v.nu = c->nu;
    v.x = c->x;
    v.wsum = c->wsum;
    v.V = c->V;
    v.ldV = c->ldA;
    v.work = c->work;
    v.ctl = c->ctl;
    v.sl = last_slot(c);
    c->cert_cut.place(&v, c->cert);
    v.dp = decide_params(p, 0);
    HIP_TRY(c, aux_certify(c->dt, v, c->cert_cut, c->stream));
    return MODAP_OK;
}

// Tuning cache: lines "dt ldA m block lanes_per_row chunks rows_per_step depth interleave grid".
const char *tune_cache_path() {
    const char *p = std::getenv("MODAP_TUNE_CACHE");
    return (p && *p) ? p : nullptr;
}

bool cache_lookup(const modap_ctx *c, modap_tile *t) {
    const char *path = tune_cache_path();
    if (!path) return false;
    FILE *f = std::fopen(path, "r");
    if (!f) return false;
    long long dt, lda, m;
    int blk, lpr, ch, rs, depth, il, grid;
    bool found = false;
    char line[256];
    while (std::fgets(line, sizeof line, f)) {
        if (std::sscanf(line, "%lld %lld %lld %d %d %d %d %d %d %d", &dt, &lda, &m, &blk, &lpr, &ch, &rs, &depth,
                        &il, &grid) != 10)
            continue;  // not a line of this format
        if (dt == c->dt && lda == c->ldA && m == c->m) {  // the last matching line wins
            t->kind = 0;
            t->block = blk;
            t->lanes_per_row = lpr;
            t->chunks = ch;
            t->rows_per_step = rs;
            t->depth = depth;
            t->interleave = il;
            t->grid = grid;
            found = true;
        }
    }
    std::fclose(f);
    return found;
}

void cache_store(const modap_ctx *c, const modap_tile &t) {
    const char *path = tune_cache_path();
    if (!path) return;
    FILE *f = std::fopen(path, "a");
    if (!f) return;
    std::fprintf(f, "%d %lld %lld %d %d %d %d %d %d %d\n", c->dt, (long long)c->ldA, (long long)c->m, t.block,
                 t.lanes_per_row, t.chunks, t.rows_per_step, t.depth, t.interleave, t.grid);
    std::fclose(f);
}

// A new system.  `owned`, if given, is A in device memory with rows of the
// padded length (zeros past n); it becomes the context's on success.
modap_status set_system(modap_ctx *c, int64_t m, int64_t n, modap_dtype storage, const void *A, int64_t lda,
                        const double *b, const double *x0, int on_dev, void *owned) {
    modap_status st = check_ctx(c, false);
    if (st) return st;
    const char *msg = nullptr;
    if ((st = check_system(m, n, lda, A, b, (int)storage, &msg))) return fail(c, st, msg);
    if (!on_dev) {
        if (!all_finite(b, m)) return fail(c, MODAP_E_INVAL, "b has a non-finite entry");
        if (x0 && !all_finite(x0, n)) return fail(c, MODAP_E_INVAL, "x0 has a non-finite entry");
    }
    DeviceGuard g(c->device);
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    release_system(c);
    c->dt = (int)storage;
    c->es = elem_size(c->dt);
    c->m = m;
    c->n = n;
    const int64_t v = vec_elems(c->dt);
    c->ldA = (n + v - 1) / v * v;
    c->vpend_maybe = false;
    c->jn = 0;
    const size_t abytes = (size_t)m * (size_t)c->ldA * c->es;
    struct Adopted {   // an adopted A stays the caller's until the call succeeds
        modap_ctx *c;
        bool held;
        ~Adopted() {
            if (held) c->A = nullptr;
        }
    } adopted{c, owned != nullptr};
    if (owned)
        c->A = owned;
    else
        HIP_TRY(c, hipMalloc(&c->A, abytes));
    // x, y, the one-shot translation and the evaluation point are padded with
    // zeros to ldA so that the sweep reads whole 16-byte vectors of them.
    const size_t vbytes = sizeof(double) * (size_t)c->ldA, wbytes = 3 * acc_size(c->dt) * (size_t)c->ldA;
    Pieces pc;
    pc.add(c->x, vbytes);
    pc.add(c->y, vbytes);
    pc.add(c->vpend, vbytes);
    pc.add(c->wsum, vbytes);
    pc.add(c->x_eval, vbytes);
    pc.add(c->y_eval, vbytes);
    pc.add(c->work, wbytes);
    pc.add(c->work_eval, wbytes);
    pc.add(c->claim, sizeof(int) * m);
    const size_t zeros = pc.total;   // everything so far starts as zeros
    pc.add(c->b, sizeof(double) * m);
    pc.add(c->bref, sizeof(double) * m);
    pc.add(c->nu, sizeof(double) * m);
    pc.add(c->r_eval, sizeof(double) * m);
    pc.add(c->ynp, sizeof(double) * (size_t)reduce_grid(c));
    HIP_TRY(c, pc.alloc(c->vectors));
    HIP_TRY(c, hipMemsetAsync(c->vectors, 0, zeros, c->stream));
    if (!owned) {
        if (c->ldA != n) HIP_TRY(c, hipMemsetAsync(c->A, 0, abytes, c->stream));
        HIP_TRY(c, hipMemcpy2DAsync(c->A, (size_t)c->ldA * c->es, A, (size_t)lda * c->es, (size_t)n * c->es, (size_t)m,
                                    on_dev ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice, c->stream));
    }
    if ((st = to_device(c, c->b, b, sizeof(double) * m, on_dev))) return st;
    if (x0 && (st = to_device(c, c->x, x0, sizeof(double) * n, on_dev))) return st;
    HIP_TRY(c, hipMemcpyAsync(c->bref, c->b, sizeof(double) * m, hipMemcpyDeviceToDevice, c->stream));
    HIP_TRY(c, aux_ctl_init(c->ctl, c->checks, c->stream));
    HIP_TRY(c, aux_row_norms(c->dt, c->A, c->ldA, m, n, c->nu, &c->checks->bad, c->stream));
    if (on_dev) HIP_TRY(c, aux_check_finite(c->b, m, c->x, n, &c->checks->flag, c->stream));
    HIP_TRY(c, c->rb.reserve(std::min(n, Readback::kMaxStaged)));   // for the reading of x
    DataChecks found{};
    HIP_TRY(c, read_checks(c->rb, c->checks, c->stream, &found));
    if (found.flag) {
        if (owned) c->A = nullptr;
        release_system(c);
        return fail(c, MODAP_E_INVAL, "b or x0 has a non-finite entry");
    }
    if (found.bad != ULLONG_MAX) {
        if (owned) c->A = nullptr;
        release_system(c);
        return fail(c, MODAP_E_ZERO_ROW, "row " + std::to_string(found.bad) + " is zero or not finite");
    }
    modap_tile t{};
    bool ok = false;
    if (c->tile_forced) {
        t = c->tile;
        t.grid = 0;
        ok = configure(c, t) == MODAP_OK;
    }
    if (!ok && cache_lookup(c, &t)) ok = configure(c, t) == MODAP_OK;
    if (!ok) {
        choose_shape(c->dt, c->ldA, m, c->cu_count, &t);
        c->tile_forced = false;
        if ((st = configure(c, t))) {
            if (owned) c->A = nullptr;
            release_system(c);
            return st;
        }
    }
    if ((st = plan_resident(c)) || (st = plan_relay(c))) {
        if (owned) c->A = nullptr;
        release_system(c);
        return st;
    }
    adopted.held = false;
    c->loaded = true;
    c->err.clear();
    return MODAP_OK;
}

}  // namespace

modap_status modap_adopt_system(modap_ctx *c, int64_t m, int64_t n, modap_dtype storage, void *A, const double *b,
                                const double *x0) {
    TraceRange trace_("modap_set_system");
    return set_system(c, m, n, storage, A, n, b, x0, 1, A);
}

extern "C" {

const char *modap_strerror(modap_status s) {
    switch (s) {
        case MODAP_OK: return "ok";
        case MODAP_E_INVAL: return "invalid argument";
        case MODAP_E_ZERO_ROW: return "zero or non-finite row";
        case MODAP_E_NOMEM: return "out of memory";
        case MODAP_E_DEVICE: return "device error";
        case MODAP_E_STATE: return "invalid state";
        case MODAP_E_NOT_CONVERGED: return "not converged within max_iters";
        case MODAP_E_INFEASIBLE: return "no step direction (infeasible system)";
        case MODAP_E_NUMERIC: return "non-finite value in the iteration";
        default: return "unknown status";
    }
}

const char *modap_last_error(modap_ctx *c) { return c ? c->err.c_str() : "null context"; }

modap_status modap_create(int device, void *hip_stream, modap_ctx **out) {
    if (!out) return MODAP_E_INVAL;
    *out = nullptr;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev <= 0) return MODAP_E_DEVICE;
    if (device < 0 || device >= ndev) return MODAP_E_INVAL;
    modap_ctx *c = new (std::nothrow) modap_ctx();
    if (!c) return MODAP_E_NOMEM;
    c->device = device;
    DeviceGuard g(device);
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, device) != hipSuccess) {
        delete c;
        return MODAP_E_DEVICE;
    }
    c->cu_count = prop.multiProcessorCount;
    c->stream = reinterpret_cast<hipStream_t>(hip_stream);  // NULL: the device's default stream
    Pieces pc;
    pc.add(c->ctl, sizeof(Ctrl));
    pc.add(c->tot, sizeof(Totals));
    pc.add(c->checks, sizeof(DataChecks));
    const bool ok = pc.alloc(c->small) == hipSuccess && c->rb.create(c->stream) == hipSuccess;
    if (!ok) {
        modap_destroy(c);
        return MODAP_E_NOMEM;
    }
    hipLaunchKernelGGL(ctl_init, dim3(1), dim3(64), 0, c->stream, c->ctl, c->checks);
    if (hipPeekAtLastError() != hipSuccess || hipStreamSynchronize(c->stream) != hipSuccess) {
        (void)hipGetLastError();
        modap_destroy(c);
        return MODAP_E_DEVICE;
    }
    *out = c;
    return MODAP_OK;
}

void modap_destroy(modap_ctx *c) {
    if (!c) return;
    DeviceGuard g(c->device);
    (void)hipStreamSynchronize(c->stream);
    release_system(c);
    free_dev(c->part);
    free_dev(c->pdot);
    free_dev(c->wrow);
    free_dev(c->h_part);
    free_dev(c->dmax_part);
    free_dev(c->binf_part);
    free_dev(c->small);
    free_dev(c->stage);
    c->rb.destroy();
    for (hipEvent_t e : c->events) (void)hipEventDestroy(e);
    delete c;
}

modap_status modap_set_system(modap_ctx *c, int64_t m, int64_t n, modap_dtype storage, const void *A, int64_t lda,
                              const double *b, const double *x0, int on_dev) {
    TraceRange trace_("modap_set_system");
    return set_system(c, m, n, storage, A, lda, b, x0, on_dev, nullptr);
}

modap_status modap_set_x(modap_ctx *c, const double *x, int on_dev) {
    TraceRange trace_("modap_set_x");
    modap_status st = check_ctx(c, true);
    if (st) return st;
    if (x && !on_dev && !all_finite(x, c->n)) return fail(c, MODAP_E_INVAL, "x has a non-finite entry");
    DeviceGuard g(c->device);
    if (x) {
        if ((st = to_device(c, c->x, x, sizeof(double) * c->n, on_dev))) return st;
    } else {
        HIP_TRY(c, hipMemsetAsync(c->x, 0, sizeof(double) * c->ldA, c->stream));
    }
    hipLaunchKernelGGL(ctl_restart, dim3(1), dim3(64), 0, c->stream, c->ctl, last_slot(c));
    LAUNCH_TRY(c, "ctl_restart launch");
    if (!on_dev) HIP_TRY(c, inputs_read(c->stream, {x}));
    return MODAP_OK;
}

modap_status modap_update_coeffs(modap_ctx *c, int64_t k, const int64_t *rows, const void *new_rows,
                                 const double *new_b, const double *v, int on_dev) {
    TraceRange trace_("modap_update_coeffs");
    modap_status st = check_ctx(c, true);
    if (st) return st;
    const char *msg = nullptr;
    if (k < 0 || k > c->m) return fail(c, MODAP_E_INVAL, "k out of range");
    if (k > 0 && (!rows || !new_rows || !new_b)) return fail(c, MODAP_E_INVAL, "rows, new_rows and new_b are required");
    DeviceGuard g(c->device);
    const size_t rbytes = (size_t)k * (size_t)c->n * c->es;
    if (k > 0 && !on_dev) {
        if ((st = check_rows(k, rows, new_rows, new_b, c->m, &msg))) return fail(c, st, msg);
        if ((st = check_new_rows(c->dt, new_rows, k, c->n, &msg))) return fail(c, st, msg);
    }
    if (v && !on_dev && !all_finite(v, c->n)) return fail(c, MODAP_E_INVAL, "translation has a non-finite entry");
    const int64_t *d_rows = rows;
    const void *d_new = new_rows;
    const double *d_b = new_b;
    const double *d_v = v;
    if (!on_dev) {
        const size_t o1 = 0, o2 = o1 + (size_t)k * 8, o3 = (o2 + rbytes + 15) / 16 * 16, o4 = o3 + (size_t)k * 8;
        const size_t total = o4 + (v ? (size_t)c->n * 8 : 0);
        if ((st = ensure_stage(c, total + 16))) return st;
        char *s = reinterpret_cast<char *>(c->stage);
        if (k > 0) {
            if ((st = to_device(c, s + o1, rows, (size_t)k * 8, 0))) return st;
            if ((st = to_device(c, s + o2, new_rows, rbytes, 0))) return st;
            if ((st = to_device(c, s + o3, new_b, (size_t)k * 8, 0))) return st;
        }
        if (v && (st = to_device(c, s + o4, v, (size_t)c->n * 8, 0))) return st;
        d_rows = reinterpret_cast<const int64_t *>(s + o1);
        d_new = s + o2;
        d_b = reinterpret_cast<const double *>(s + o3);
        d_v = v ? reinterpret_cast<const double *>(s + o4) : nullptr;
    }
    if (k > 0 && on_dev) HIP_TRY(c, aux_claim_rows(d_rows, k, c->m, c->claim, c->ctl, last_slot(c), c->stream));
    if (k > 0 && (st = launch_scatter(c, k, d_rows, d_new, d_b))) return st;
    if (k > 0 && on_dev) HIP_TRY(c, aux_release_rows(d_rows, k, c->m, c->claim, c->stream));
    if (d_v) {
        hipLaunchKernelGGL(vpend_add, dim3(1), dim3(1024), 0, c->stream, c->ctl, last_slot(c), c->vpend, d_v, c->n);
        LAUNCH_TRY(c, "vpend_add launch");
        c->vpend_maybe = true;
    }
    if (!on_dev && k > 0) HIP_TRY(c, inputs_read(c->stream, {rows, new_rows, new_b}));
    if (!on_dev) HIP_TRY(c, inputs_read(c->stream, {v}));
    return MODAP_OK;
}

modap_status modap_set_drift(modap_ctx *c, int64_t T, const double *V, int64_t ldv, int on_dev) {
    TraceRange trace_("modap_set_drift");
    modap_status st = check_ctx(c, true);
    if (st) return st;
    const char *msg = nullptr;
    if ((st = check_drift(T, V, ldv, c->n, !on_dev, &msg))) return fail(c, st, msg);
    DeviceGuard g(c->device);
    if (under_capture(c)) return hip_fail(c, hipErrorStreamCaptureUnsupported, "modap_set_drift");
    const int sl = last_slot(c);
    if (c->V) {
        hipLaunchKernelGGL(sched_to_vpend, dim3(1), dim3(1024), 0, c->stream, c->ctl, sl, c->vpend,
                           (const double *)c->V, c->ldA, c->n);
        LAUNCH_TRY(c, "sched_to_vpend launch");
        c->vpend_maybe = true;
    }
    c->T = 0;
    const size_t want = T > 0 && V ? (size_t)T * (size_t)c->ldA : 0;
    if (!want || want > c->V_cap || want < c->V_cap / 4) {   // (the kept schedule is at most four times what is needed)
        HIP_TRY(c, hipStreamSynchronize(c->stream));
        free_dev(c->V);
        c->V_cap = 0;
        if (want) HIP_TRY(c, hipMalloc(&c->V, sizeof(double) * want));
        c->V_cap = want;
    }
    if (!want) {
        hipLaunchKernelGGL(ctl_set_drift, dim3(1), dim3(64), 0, c->stream, c->ctl, sl, (int64_t)0);
        LAUNCH_TRY(c, "ctl_set_drift launch");
        return MODAP_OK;
    }
    // rows padded with zeros to ldA, like x
    auto take_in = [&]() -> modap_status {
        if (on_dev) {
            const int64_t work = T * ((c->ldA + kDriftCols - 1) / kDriftCols);
            hipLaunchKernelGGL(drift_in, dim3((unsigned)std::min<int64_t>(work, kDriftGroups)), dim3(256), 0, c->stream,
                               V, ldv, c->n, T, c->V, c->ldA, &c->checks->flag, c->ctl, sl, c->rb.dev, c->rb.arrived,
                               ++c->rb.seq);
            LAUNCH_TRY(c, "drift_in launch");
            HIP_TRY(c, c->rb.wait(c->stream));
            return c->rb.view->fault ? fail(c, MODAP_E_INVAL, "drift has a non-finite entry") : MODAP_OK;
        }
        if (c->ldA != c->n) HIP_TRY(c, hipMemsetAsync(c->V, 0, sizeof(double) * want, c->stream));
        HIP_TRY(c, hipMemcpy2DAsync(c->V, sizeof(double) * c->ldA, V, sizeof(double) * ldv, sizeof(double) * c->n,
                                    (size_t)T, hipMemcpyHostToDevice, c->stream));
        hipLaunchKernelGGL(ctl_set_drift, dim3(1), dim3(64), 0, c->stream, c->ctl, sl, T);
        LAUNCH_TRY(c, "ctl_set_drift launch");
        // (a copy from pinned memory waits in the stream, behind whatever is
        // queued there, and V is the caller's again when the call returns)
        HIP_TRY(c, hipStreamSynchronize(c->stream));
        return MODAP_OK;
    };
    if ((st = take_in())) {   // no schedule is left behind
        free_dev(c->V);
        c->V_cap = 0;
        return st;
    }
    c->T = T;
    return MODAP_OK;
}

modap_status modap_iterate(modap_ctx *c, const modap_params *p, int64_t k, modap_stats *out) {
    TraceRange trace_("modap_iterate");
    modap_status st = check_ctx(c, true);
    if (st) return st;
    if ((st = check_params(c, p))) return st;
    if (k < 0) return fail(c, MODAP_E_INVAL, "k < 0");
    DeviceGuard g(c->device);
    const auto t0 = std::chrono::steady_clock::now();
    hipLaunchKernelGGL(ctl_begin, dim3(1), dim3(64), 0, c->stream, c->ctl, last_slot(c), (int64_t)-1);
    LAUNCH_TRY(c, "ctl_begin launch");
    size_t ev = 0;
    double bytes = 0.0;
    const int track = p->track != 0;
    if (use_resident(c, p)) {
        // one launch of many iterations (each launch settles its own checks)
        for (int64_t done = 0; done < k;) {
            const int64_t K = std::min<int64_t>(k - done, int64_t(1) << 20);
            if ((st = launch_resident(c, p, track, K, nullptr, &bytes))) return st;
            done += K;
        }
    } else {
        if ((st = enqueue_prime(c, c->work, c->x))) return st;
        if ((st = reserve_events(c, k, p->profile))) return st;
        for (int64_t i = 0; i < k; ++i)
            if ((st = enqueue_iteration(c, p, track, i, nullptr, &ev, &bytes))) return st;
        if (k > 0 && (st = enqueue_settle(c, p, track))) return st;
    }
    // (a tracked iteration never stops: there is nothing to certify)
    const bool certify = k > 0 && p->certify && !track;
    if (!out) return certify ? enqueue_certify(c, p) : MODAP_OK;
    State kc;
    if ((st = read_back(c, &kc))) return st;
    if (certify && kc.status == ST_CONVERGED && !kc.certified) {
        if ((st = enqueue_certify(c, p))) return st;
        if ((st = read_back(c, &kc))) return st;
    }
    if (p->profile) HIP_TRY(c, hipStreamSynchronize(c->stream));   // the events too
    *out = modap_stats{};
    fill_stats(out, kc);
    out->seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    out->hbm_bytes = bytes;
    out->resident = use_resident(c, p) ? 1 : 0;
    if (p->profile && (st = profile_totals(c, ev, out))) return st;
    if (!kc.vpend_valid && kc.v_idx < 0) c->vpend_maybe = false;
    return status_of(c, kc, false);
}

modap_status modap_solve(modap_ctx *c, const modap_params *p, modap_stats *out) {
    TraceRange trace_("modap_solve");
    modap_status st = check_ctx(c, true);
    if (st) return st;
    if ((st = check_params(c, p))) return st;
    DeviceGuard g(c->device);
    const auto t0 = std::chrono::steady_clock::now();
    hipLaunchKernelGGL(ctl_begin, dim3(1), dim3(64), 0, c->stream, c->ctl, last_slot(c), (int64_t)p->max_iters);
    LAUNCH_TRY(c, "ctl_begin launch");
    const bool resident = use_resident(c, p);
    if (!resident && (st = enqueue_prime(c, c->work, c->x))) return st;
    const int64_t total = p->max_iters + 1;  // the last sweep checks the last step
    if (!resident && (st = reserve_events(c, std::min<int64_t>(total, 4096), p->profile))) return st;
    size_t ev = 0;
    double bytes = 0.0;
    auto observed = t0;
    State kc;
    // Passes of queued iterations until the device stops; a stop at
    // eps-feasibility that the FP64 certificate does not confirm has taken a
    // step instead, and the next pass goes on from there.  The step limit is
    // the device's, so a pass may queue more iterations than remain.
    int64_t ahead = resident ? 0 : solve_ahead(c);
    for (;;) {
        // Each sweep tells the host the decision it takes on the previous
        // check (a resident launch its last one).  The host keeps a few
        // iterations (two launches) queued beyond the last decision it has
        // seen, so the device never waits for it and few are queued in vain.
        const int64_t first = c->jn;
        int64_t queued = 0, chunk = 16, settled = 0;
        int64_t prev_end = first - 1, last_end = first - 1;   // last checks of the two newest resident launches
        uint32_t idle = 0;
        bool stopped = false;
        volatile uint64_t *word = &c->rb.view->progress;
        *word = 0;   // (nothing that writes it is queued)
        auto look = [&]() {
            const uint64_t w = *word;
            if (w == 0) return;
            stopped = (w & 0xff) != ST_RUNNING;
            const int64_t now_settled = (int64_t)(w >> 8) - first;
            if (now_settled != settled) idle = 0;
            settled = now_settled;
            ahead = solve_ahead_after(ahead, queued - settled, settled);
        };
        auto room = [&]() { return resident ? first - 1 + settled >= prev_end : queued - settled < ahead; };
        while (queued < total && !stopped) {
            // a chunk: what there is room for, and the wait until there is more
            TraceRange trace_chunk("modap_solve chunk");
            do {
                if (resident) {
                    const int64_t cnt = std::min(chunk, total - queued);
                    if ((st = launch_resident(c, p, 0, cnt, &c->rb.dev->progress, &bytes))) return st;
                    queued += cnt;
                    prev_end = last_end;
                    last_end = c->jn - 1;
                    chunk = std::min<int64_t>(chunk * 2, 1024);
                } else {
                    if ((st = enqueue_iteration(c, p, 0, queued, &c->rb.dev->progress, &ev, &bytes))) return st;
                    ++queued;
                }
            } while (queued < total && room());
            for (look(); queued < total && !stopped && !room(); look())
                if ((st = poll_pause(c, ++idle))) return st;
        }
        if (!resident && (st = enqueue_settle(c, p, 0))) return st;
        if ((st = read_back(c, &kc))) return st;
        observed = std::chrono::steady_clock::now();
        if (!(p->certify && kc.status == ST_CONVERGED && !kc.certified)) break;
        if ((st = enqueue_certify(c, p))) return st;
        if ((st = read_back(c, &kc))) return st;
        bytes += sweep_bytes(c, false);
        observed = std::chrono::steady_clock::now();
        if (kc.status != ST_RUNNING) break;
    }
    if (p->profile) HIP_TRY(c, hipStreamSynchronize(c->stream));   // the events too
    if (out) {
        *out = modap_stats{};
        fill_stats(out, kc);
        out->seconds = std::chrono::duration<double>(observed - t0).count();
        out->hbm_bytes = bytes;
        out->resident = resident ? 1 : 0;
        if (p->profile && (st = profile_totals(c, ev, out))) return st;
    }
    if (!kc.vpend_valid && kc.v_idx < 0) c->vpend_maybe = false;
    if (kc.status == ST_RUNNING) return fail(c, MODAP_E_NOT_CONVERGED, "step limit reached before eps-feasibility");
    return status_of(c, kc, true);
}

constexpr int64_t kAnnounceGroups = 32;
modap_status modap_eval_sweep(modap_ctx *c, const double *x, double *r, double *y, int64_t *h, double *max_viol,
                              int on_dev) {
    TraceRange trace_("modap_eval_sweep");
    modap_status st = check_ctx(c, true);
    if (st) return st;
    if (!x || !y) return fail(c, MODAP_E_INVAL, "x and y are required");
    DeviceGuard g(c->device);
    // The point is read, and device results are written, where the caller
    // holds them; host ones pass through the staging memory.
    const int64_t nr = r ? c->m : 0;
    const bool staged = !on_dev && c->n + nr <= Readback::kMaxStaged;
    if (on_dev) {
        if ((st = enqueue_prime(c, c->work_eval, x))) return st;
    } else {
        if ((st = to_device(c, c->x_eval, x, sizeof(double) * c->n, 0))) return st;
        if ((st = enqueue_prime(c, c->work_eval, c->x_eval))) return st;
    }
    const bool hv = translation_possible(c);
    SweepArgs a = sweep_args(c);
    a.b_out = nullptr;
    a.work = c->work_eval;
    a.check_status = 0;
    a.r_out = !r ? nullptr : on_dev ? r : c->r_eval;
    if ((st = launch_sweep(c, a, hv, nullptr, nullptr))) return st;
    ReduceArgs ra = reduce_args(c);
    ra.y = on_dev ? y : c->y_eval;
    ra.ctl = nullptr;
    ra.iterate = 0;
    // Results that stay on the device leave only the totals to tell: the
    // reduction does it itself, up to kAnnounceGroups workgroups (each waits
    // for its writes to reach the host's view: a 50 x 200 evaluation takes
    // 24.8 us, and 26.2 with a launch that publishes).
    const bool told = on_dev && reduce_grid(c) <= kAnnounceGroups;
    if (told) {
        ra.view = c->rb.dev;
        ra.fault = &c->ctl->fault;
        ra.arrived = c->rb.arrived;
        ra.seq = ++c->rb.seq;
    }
    if ((st = launch_reduce(c, ra))) return st;
    PublishArgs pa{};
    pa.tot = c->tot;
    pa.fault = &c->ctl->fault;
    if (told) {
        HIP_TRY(c, c->rb.wait(c->stream));
    } else if (staged) {
        HIP_TRY(c, c->rb.reserve(c->n + nr));
        pa.src[0] = c->y_eval;
        pa.src[1] = c->r_eval;
        pa.dst[0] = c->rb.buf_dev;
        pa.dst[1] = c->rb.buf_dev + c->n;
        pa.count[0] = c->n;
        pa.count[1] = nr;
    } else if (!on_dev) {
        if ((st = from_device(c, y, c->y_eval, sizeof(double) * c->n, 0))) return st;
        if (r && (st = from_device(c, r, c->r_eval, sizeof(double) * c->m, 0))) return st;
    }
    if (!told) HIP_TRY(c, c->rb.run(pa, c->stream));
    if (staged) {
        std::memcpy(y, c->rb.buf, sizeof(double) * (size_t)c->n);
        if (r) std::memcpy(r, c->rb.buf + c->n, sizeof(double) * (size_t)c->m);
    }
    if (c->rb.view->fault) return fault_status(c);
    const Totals to = c->rb.view->tot;
    if (h) *h = to.h;
    if (max_viol) *max_viol = to.dmax;
    return MODAP_OK;
}

modap_status modap_query(modap_ctx *c, double *x, double *b, modap_stats *out, int on_dev) {
    TraceRange trace_("modap_query");
    modap_status st = check_ctx(c, true);
    if (st) return st;
    DeviceGuard g(c->device);
    // the right-hand side is the data as the caller sees them, every
    // translation applied, in FP64; nothing is committed, so reading b does
    // not change the iteration
    if (b)
        HIP_TRY(c, aux_rhs_exact(c->dt, c->A, c->ldA, c->m, c->n, c->ctl, last_slot(c), c->bref, c->wsum, c->vpend,
                                 c->V, c->ldA, on_dev ? b : c->r_eval, c->stream));
    State kc;
    if (on_dev) {
        if (x && (st = from_device(c, x, c->x, sizeof(double) * c->n, 1))) return st;
        st = read_back(c, &kc);
    } else {
        st = read_back(c, &kc, c->x, x, x ? c->n : 0, c->r_eval, b, b ? c->m : 0);
    }
    if (st) return st;
    if (out) {
        *out = modap_stats{};
        fill_stats(out, kc);
    }
    return MODAP_OK;
}

modap_status modap_set_tile(modap_ctx *c, const modap_tile *t) {
    if (!c) return MODAP_E_INVAL;
    DeviceGuard g(c->device);
    if (!t) {
        c->tile_forced = false;
        if (!c->loaded) return MODAP_OK;
        modap_tile d{};
        choose_shape(c->dt, c->ldA, c->m, c->cu_count, &d);
        HIP_TRY(c, hipStreamSynchronize(c->stream));
        return configure(c, d);
    }
    if (!c->loaded) {
        c->tile = *t;
        c->tile_forced = true;
        return MODAP_OK;
    }
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    const modap_tile keep = c->tile;
    modap_status st = configure(c, *t);
    if (st) {
        const std::string msg = c->err;
        (void)configure(c, keep);
        return fail(c, st, msg);
    }
    c->tile_forced = true;
    return MODAP_OK;
}

modap_status modap_autotune(modap_ctx *c, int reps, modap_tile *best) {
    TraceRange trace_("modap_autotune");
    modap_status st = check_ctx(c, true);
    if (st) return st;
    if (reps < 1) return fail(c, MODAP_E_INVAL, "reps < 1");
    DeviceGuard g(c->device);
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    const modap_tile keep = c->tile;
    const bool hv = translation_possible(c);
    if (!event_at(c, 2 * (size_t)reps - 1)) return fail(c, MODAP_E_DEVICE, "hipEventCreate failed");
    if ((st = enqueue_prime(c, c->work_eval, c->x))) return st;
    int cnt = 0;
    const SweepKernel *tab = kernels_for(c->dt, &cnt);
    modap_tile win = keep;
    float win_ms = 1e30f;
    std::vector<float> times;
    // The built-in shape is timed first, and a challenger must beat the
    // incumbent by kMargin: near-equal shapes do not flip with timing noise.
    constexpr float kMargin = 0.98f;
    std::vector<modap_tile> order;
    modap_tile def{};
    choose_shape(c->dt, c->ldA, c->m, c->cu_count, &def);
    if (def.kind == 0) order.push_back(def);
    for (int i = 0; i < cnt; ++i) {
        if (tab[i].has_v != hv) continue;
        if (coverage(c->dt, tab[i].lpr, tab[i].chunks) < c->ldA) continue;
        int per_cu = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, tab[i].func, tab[i].block, 0) != hipSuccess ||
            per_cu < 1)
            per_cu = 1;
        for (int trial = 0; trial < 2 * std::max(2, per_cu); ++trial) {
            const int mult = trial / 2 + 1, il = trial % 2;
            modap_tile t{0, tab[i].block, tab[i].lpr, tab[i].chunks, c->cu_count * mult, tab[i].rs, tab[i].pd, il};
            if (mult > 1 && mult != per_cu && mult != 2) continue;
            order.push_back(t);
        }
    }
    for (const modap_tile &t : order) {
        if (configure(c, t) != MODAP_OK) continue;
        SweepArgs a = sweep_args(c);
        a.b_out = nullptr;
        a.work = c->work_eval;
        a.check_status = 0;
        const SweepKernel *k = hv ? c->kern_v : c->kern_nov;
        // an untimed sweep, then `reps` timed ones back to back (as the
        // iterations run; a host wait after each would leave the device idle
        // between them); the shortest counts, the work being the same each time
        HIP_TRY(c, k->launch(a, c->tile.grid, c->stream, nullptr, nullptr));
        for (int r = 0; r < reps; ++r)
            HIP_TRY(c, k->launch(a, c->tile.grid, c->stream, event_at(c, 2 * (size_t)r), event_at(c, 2 * (size_t)r + 1)));
        HIP_TRY(c, hipEventSynchronize(event_at(c, 2 * (size_t)reps - 1)));
        times.clear();
        for (int r = 0; r < reps; ++r) {
            float ms = 0.f;
            HIP_TRY(c, hipEventElapsedTime(&ms, event_at(c, 2 * (size_t)r), event_at(c, 2 * (size_t)r + 1)));
            times.push_back(ms);
        }
        const float best_ms = *std::min_element(times.begin(), times.end());
        if (best_ms < win_ms * kMargin || win_ms == 1e30f) {
            win_ms = best_ms;
            win = c->tile;
        }
        HIP_TRY(c, hipStreamSynchronize(c->stream));
    }
    if ((st = configure(c, win))) {
        (void)configure(c, keep);
        return st;
    }
    if (c->tile.kind == 0) c->tile_forced = true;   // (rows too long for a one-pass shape: nothing was timed)
    cache_store(c, c->tile);
    if (best) *best = c->tile;
    return MODAP_OK;
}

modap_status modap_get_tile(modap_ctx *c, modap_tile *t) {
    modap_status st = check_ctx(c, true);
    if (st) return st;
    if (!t) return fail(c, MODAP_E_INVAL, "tile is NULL");
    *t = c->tile;
    return MODAP_OK;
}

}  // extern "C"

// Launchers of the auxiliary kernels for the other translation units.
namespace modap {

hipError_t aux_row_norms(int dt, const void *A, int64_t ldA, int64_t m, int64_t n, double *nu,
                         unsigned long long *bad, hipStream_t s) {
    const int nb = (int)((m + 3) / 4);
    switch (dt) {
        case 0: hipLaunchKernelGGL(row_norms<0>, dim3(nb), dim3(256), 0, s, A, ldA, m, n, nu, bad); break;
        case 1: hipLaunchKernelGGL(row_norms<1>, dim3(nb), dim3(256), 0, s, A, ldA, m, n, nu, bad); break;
        default: hipLaunchKernelGGL(row_norms<2>, dim3(nb), dim3(256), 0, s, A, ldA, m, n, nu, bad); break;
    }
    return hipGetLastError();
}

hipError_t aux_check_finite(const double *p, int64_t np, const double *q, int64_t nq, unsigned long long *flag,
                            hipStream_t s) {
    hipLaunchKernelGGL(check_finite, dim3(64), dim3(256), 0, s, p, np, q, nq, flag);
    return hipGetLastError();
}

hipError_t aux_ctl_init(Ctrl *c, DataChecks *checks, hipStream_t s) {
    hipLaunchKernelGGL(ctl_init, dim3(1), dim3(64), 0, s, c, checks);
    return hipGetLastError();
}

hipError_t aux_scatter_rows(int dt, void *A, int64_t ldA, int64_t m, int64_t n, int64_t k, const int64_t *rows,
                            const void *new_rows, const double *new_b, double *b, double *bref, double *nu, Ctrl *ctl,
                            int sl, const double *vpend, const double *V, int64_t ldV, const double *wsum,
                            hipStream_t s) {
    switch (dt) {
        case 0: hipLaunchKernelGGL(scatter_rows<0>, dim3(k), dim3(256), 0, s, A, ldA, m, n, rows, new_rows, new_b, b, bref, nu, ctl, sl, vpend, V, ldV, wsum); break;
        case 1: hipLaunchKernelGGL(scatter_rows<1>, dim3(k), dim3(256), 0, s, A, ldA, m, n, rows, new_rows, new_b, b, bref, nu, ctl, sl, vpend, V, ldV, wsum); break;
        default: hipLaunchKernelGGL(scatter_rows<2>, dim3(k), dim3(256), 0, s, A, ldA, m, n, rows, new_rows, new_b, b, bref, nu, ctl, sl, vpend, V, ldV, wsum); break;
    }
    return hipGetLastError();
}

hipError_t aux_claim_rows(const int64_t *rows, int64_t k, int64_t m, int *claim, Ctrl *ctl, int sl, hipStream_t s) {
    const int grid = (int)std::min<int64_t>(1024, (k + 255) / 256);
    hipLaunchKernelGGL(claim_rows, dim3(grid), dim3(256), 0, s, rows, k, m, claim, ctl, sl);
    return hipGetLastError();
}

hipError_t aux_release_rows(const int64_t *rows, int64_t k, int64_t m, int *claim, hipStream_t s) {
    const int grid = (int)std::min<int64_t>(1024, (k + 255) / 256);
    hipLaunchKernelGGL(release_rows, dim3(grid), dim3(256), 0, s, rows, k, m, claim);
    return hipGetLastError();
}

hipError_t aux_vpend_add(Ctrl *c, int sl, double *vpend, const double *v, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(vpend_add, dim3(1), dim3(1024), 0, s, c, sl, vpend, v, n);
    return hipGetLastError();
}

hipError_t aux_sched_to_vpend(Ctrl *c, int sl, double *vpend, const double *V, int64_t ldV, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(sched_to_vpend, dim3(1), dim3(1024), 0, s, c, sl, vpend, V, ldV, n);
    return hipGetLastError();
}

hipError_t aux_ctl_set_drift(Ctrl *c, int sl, int64_t T, hipStream_t s) {
    hipLaunchKernelGGL(ctl_set_drift, dim3(1), dim3(64), 0, s, c, sl, T);
    return hipGetLastError();
}

hipError_t aux_rhs_exact(int dt, const void *A, int64_t ldA, int64_t m, int64_t n, const Ctrl *ctl, int sl,
                         const double *bref, const double *wsum, const double *vpend, const double *V, int64_t ldV,
                         double *out, hipStream_t s) {
    const int nb = (int)((m + 4 * kRows64 - 1) / (4 * kRows64));
    switch (dt) {
        case 0: hipLaunchKernelGGL(rhs_exact<0>, dim3(nb), dim3(256), 0, s, A, ldA, m, n, ctl, sl, bref, wsum, vpend, V, ldV, out); break;
        case 1: hipLaunchKernelGGL(rhs_exact<1>, dim3(nb), dim3(256), 0, s, A, ldA, m, n, ctl, sl, bref, wsum, vpend, V, ldV, out); break;
        default: hipLaunchKernelGGL(rhs_exact<2>, dim3(nb), dim3(256), 0, s, A, ldA, m, n, ctl, sl, bref, wsum, vpend, V, ldV, out); break;
    }
    return hipGetLastError();
}

bool static_sweep_plan(int dt, int64_t ldA, int64_t m, int64_t n, int cu_count, int per_cu, StaticPlan *out) {
    modap_tile t{};
    choose_shape(dt, ldA, m, cu_count, &t);
    // (FP64 rows above 4096 elements have a one-pass shape, whose partials do
    // not always fit the static scratch: they stay refused)
    if (t.kind != 0 || (dt == 0 && ldA > 4096)) return false;
    const SweepKernel *k = find_kernel(dt, t.block, t.lanes_per_row, t.chunks, t.rows_per_step, t.depth, false);
    if (!k) return false;
    // the row mapping of configure() for a band of rows per workgroup
    const int per_step = (t.block / t.lanes_per_row) * t.rows_per_step;
    int grid = std::min(t.grid > 0 ? t.grid : std::max(1, cu_count), per_cu * std::max(1, cu_count));
    int64_t rpb = (m + grid - 1) / grid;
    rpb = ((rpb + per_step - 1) / per_step) * per_step;
    grid = (int)((m + rpb - 1) / rpb);
    out->k = k;
    out->grid = grid;
    out->R = (int)((n + 63) / 64);
    out->cov = coverage(dt, t.lanes_per_row, t.chunks);
    out->rows_per_block = rpb;
    out->block_stride = rpb;
    out->step_stride = per_step;
    return true;
}

hipError_t static_sweep_launch(int dt, const StaticPlan &plan, const SweepScratch &s, const void *A, int64_t ldA,
                               int64_t m, int64_t n, const double *b, const double *x, double *r, double *y,
                               int64_t *h, double *max_viol, hipStream_t stream) {
    const int nb = (int)((m + 3) / 4), sg = (int)std::min<int64_t>(1024, (ldA + 255) / 256);
    switch (dt) {
        case 0: hipLaunchKernelGGL(static_begin<0>, dim3(nb + sg), dim3(256), 0, stream, A, ldA, m, n, s.nu, s.bad, x, s.work, s.ctl, nb); break;
        case 1: hipLaunchKernelGGL(static_begin<1>, dim3(nb + sg), dim3(256), 0, stream, A, ldA, m, n, s.nu, s.bad, x, s.work, s.ctl, nb); break;
        default: hipLaunchKernelGGL(static_begin<2>, dim3(nb + sg), dim3(256), 0, stream, A, ldA, m, n, s.nu, s.bad, x, s.work, s.ctl, nb); break;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    SweepArgs a{};
    a.A = A;
    a.ldA = ldA;
    a.m = m;
    a.n = n;
    a.b_in = b;
    a.b_out = nullptr;
    a.nu = s.nu;
    a.work = s.work;
    a.pd.ctl = s.ctl;
    a.pd.j = 1;          // runs under the fresh state in slot 0
    a.pd.decide = 0;
    a.check_status = 0;
    a.r_out = r;
    a.part = s.part;
    a.ldPart = plan.cov;
    a.h_part = s.h_part;
    a.dmax_part = s.dmax_part;
    a.binf_part = s.binf_part;
    a.rows_per_block = plan.rows_per_block;
    a.block_stride = plan.block_stride;
    a.step_stride = plan.step_stride;
    if ((e = plan.k->launch(a, plan.grid, stream, nullptr, nullptr)) != hipSuccess) return e;
    ReduceArgs ra{};
    ra.part = s.part;
    ra.ldPart = plan.cov;
    ra.G = plan.grid;
    ra.acc_f64 = dt == 0;
    ra.Gs = plan.grid;
    ra.n = n;
    ra.ldA = ldA;
    ra.y = y;
    ra.h_part = s.h_part;
    ra.dmax_part = s.dmax_part;
    ra.binf_part = s.binf_part;
    ra.tot = s.tot;
    ra.ynp = s.ynp;
    ra.h_out = h;
    ra.dmax_out = max_viol;
    if (dt == 0)
        hipLaunchKernelGGL(reduce_y<double>, dim3(plan.R), dim3(kReduceThreads), 0, stream, ra);
    else
        hipLaunchKernelGGL(reduce_y<float>, dim3(plan.R), dim3(kReduceThreads), 0, stream, ra);
    return hipGetLastError();
}

CertPlan cert_plan(int dt, int64_t m, int64_t n, int64_t ldA, int64_t workgroups) {
    CertPlan p{};
    const int64_t groups = (m + kCertGroup - 1) / kCertGroup, tile = 256 * (int64_t)vec_elems(dt);
    p.Gs = (int)std::max<int64_t>(1, std::min(groups, workgroups));
    p.rows_per_band = std::max<int64_t>(256, (m + 127) / 128);   // at most 128 bands: their partials are FP64 rows
    p.bands = (int)((m + p.rows_per_band - 1) / p.rows_per_band);
    p.tiles = (int)((ldA + tile - 1) / tile);
    p.R = (int)((n + 63) / 64);
    auto up = [](size_t v) { return (v + 255) & ~(size_t)255; };
    p.bytes = up(8 * (size_t)m) + up(8 * (size_t)p.bands * (size_t)ldA) + up(8 * (size_t)ldA) + up(8 * (size_t)p.R) +
              4 * up(8 * (size_t)p.Gs) + up(4 * (size_t)p.bands) + up(sizeof(Totals));
    return p;
}

void CertPlan::place(CertArgs *a, void *base) const {
    unsigned char *at = static_cast<unsigned char *>(base);
    auto take = [&](size_t bytes) {
        unsigned char *q = at;
        at += (bytes + 255) & ~(size_t)255;
        return q;
    };
    a->wt = reinterpret_cast<double *>(take(8 * (size_t)a->m));
    a->part = reinterpret_cast<double *>(take(8 * (size_t)bands * (size_t)a->ldA));
    a->y = reinterpret_cast<double *>(take(8 * (size_t)a->ldA));
    a->ynp = reinterpret_cast<double *>(take(8 * (size_t)R));
    a->h_part = reinterpret_cast<int64_t *>(take(8 * (size_t)Gs));
    a->dmax_part = reinterpret_cast<double *>(take(8 * (size_t)Gs));
    a->binf_part = reinterpret_cast<double *>(take(8 * (size_t)Gs));
    a->drift_part = reinterpret_cast<double *>(take(8 * (size_t)Gs));
    a->band_rows = reinterpret_cast<int32_t *>(take(4 * (size_t)bands));
    a->tot = reinterpret_cast<Totals *>(take(sizeof(Totals)));
    a->R = R;
    a->Gs = Gs;
    a->bands = bands;
    a->rows_per_band = rows_per_band;
}

template <int DT>
static void launch_cert(const CertArgs &a, const CertPlan &p, hipStream_t s) {
    using Acc = typename Store<DT>::Acc;
    const CertArgs *nl = nullptr;
    const CertJob *nj = nullptr;
    hipLaunchKernelGGL(cert_dot<DT>, dim3(p.Gs), dim3(256), 0, s, a, nl, nj);
    hipLaunchKernelGGL(cert_axpy<DT>, dim3(p.bands, p.tiles), dim3(256), 0, s, a, nl, nj);
    hipLaunchKernelGGL(cert_reduce, dim3(p.R), dim3(256), 0, s, a, nl, nj);
    hipLaunchKernelGGL(cert_decide<Acc>, dim3(1), dim3(1024), 0, s, a, nl);
}

template <int DT>
static void launch_cert_list(const CertArgs *list, int count, const CertJob *jobs, int nd, int na, int nr, hipStream_t s) {
    using Acc = typename Store<DT>::Acc;
    const CertArgs none{};
    hipLaunchKernelGGL(cert_dot<DT>, dim3(nd), dim3(256), 0, s, none, list, jobs);
    hipLaunchKernelGGL(cert_axpy<DT>, dim3(na), dim3(256), 0, s, none, list, jobs + nd);
    hipLaunchKernelGGL(cert_reduce, dim3(nr), dim3(256), 0, s, none, list, jobs + nd + na);
    hipLaunchKernelGGL(cert_decide<Acc>, dim3(count), dim3(1024), 0, s, none, list);
}

hipError_t aux_certify(int dt, const CertArgs &a, const CertPlan &p, hipStream_t s) {
    switch (dt) {
        case 0: launch_cert<0>(a, p, s); break;
        case 1: launch_cert<1>(a, p, s); break;
        default: launch_cert<2>(a, p, s); break;
    }
    return hipGetLastError();
}

hipError_t aux_certify_list(int dt, const CertArgs *list, int count, const CertJob *jobs, int ndot, int naxpy,
                            int nreduce, hipStream_t s) {
    switch (dt) {
        case 0: launch_cert_list<0>(list, count, jobs, ndot, naxpy, nreduce, s); break;
        case 1: launch_cert_list<1>(list, count, jobs, ndot, naxpy, nreduce, s); break;
        default: launch_cert_list<2>(list, count, jobs, ndot, naxpy, nreduce, s); break;
    }
    return hipGetLastError();
}

}  // namespace modap
