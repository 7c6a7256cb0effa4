// Resident iteration for small systems: many iterations in one launch.
//
// For a system of a few MiB the two-kernel iteration (sweep, then reduction)
// is bound by latency, not bandwidth: each kernel costs a few microseconds
// whatever its size.  Here one cooperative launch of G workgroups runs K
// iterations of the method (section 3: Map of the positive slices, eq. 7,
// Reduce(+), the eq. 10 test, the step of eq. 12 or Algorithm 1, the
// translation of the data), and the workgroups meet once per iteration:
//
//   * each workgroup copies its band of rows (and their b, ||a_i||^2) into
//     LDS once, and reads them from there in every iteration;
//   * per iteration it sweeps its band (eight wavefronts, four rows at a time
//     each, lanes over the columns) and writes one partial y and its h, dmax,
//     ||b||inf to one of two sets of words (alternating by iteration), each
//     word 32 bits of data and the 32-bit number of the iteration (FP64 takes
//     two words);
//   * every workgroup reads the words of all G until they carry this
//     iteration's number, sums the partials in the same order, takes the same
//     decision and step in FP64 on its own copy of x, y and the running sum of
//     translations (identical arithmetic on identical data gives identical
//     results in every workgroup), and goes on.
// There is no barrier besides: the words are the data and their arrival in
// one.  (With partials, a release, an arrival counter that all poll and only
// then the reads -- four trips to memory in a row -- an iteration took, of
// FP64 64 x 128 4.5 us and now 3.6, 256 x 1024 5.9 and 4.9, 500 x 700 7.7 and
// 6.5; of FP32 256 x 1024 12.2 and 4.5, 400 x 1600 13.3 and 5.5: the partial
// words of 4 bytes were slow to write through.)  A workgroup writes a set
// again two iterations later: by then it has read every other workgroup's
// words of the iteration between, and each of those was written after its
// workgroup had read the set.  The numbers go on from launch to launch; where
// they would be used again (a captured launch that is replayed, 2^32 of them
// used up) the host has the words cleared before the launch.
//
// Every wait is bounded by the device's constant clock: a workgroup that
// waits longer than timeout_ticks raises ctl->fault and leaves, and so do the
// others once they see it or wait as long, so the grid always drains.  A
// launch with a fault writes nothing back (its results are void).
//
// At the end workgroup 0 writes x, y, the translation sum, the working
// vectors of the two-kernel path and the final state (into both slots); each
// workgroup writes the translated b of its band.  Semantics per iteration are
// those of the two-kernel path (check, step, data update); only the order of
// the sum over row bands differs.
#pragma once

#include <type_traits>

#include "modap_device.hpp"

namespace modap {

struct ResidentArgs {
    const void *A;          // [m x ldA] storage type
    int64_t ldA, m, n;
    int32_t ldR;            // LDS row length: n rounded up to 64 (at most 512)
    int32_t rows;           // rows per workgroup
    double *b;              // [m]
    const double *nu;       // [m]
    double *x, *y, *wsum;   // [ldA]
    const double *vpend;    // [ldA]
    const double *V;        // [T x ldV] or null
    int64_t ldV;
    void *work;             // [3 x ldA] working vectors of the two-kernel path (written at the end)
    Ctrl *ctl;
    int64_t j0;             // the launch runs under the committed state of slot (j0-1)&1
    int64_t K;              // iterations
    Decide dp;
    uint64_t *words;        // [2 x kResidentMaxGrid x resident_words(DT, ldR)]
    uint32_t base;          // number of the launch's first iteration (a set of words is cleared to number 0)
    uint64_t *progress;     // host memory or null: told the last check and its status when the launch ends
    int64_t timeout_ticks;  // constant-clock (100 MHz) ticks a workgroup waits for the others
};

// Words of one workgroup and iteration: the columns' (the low halves of all,
// then for FP64 the high halves), then h, dmax and ||b||inf.
constexpr int kTotalWords = 5;
__host__ __device__ constexpr int resident_words(int dt, int ldR) { return (dt == 0 ? 2 : 1) * ldR + kTotalWords; }
// All words of a context: two sets of the workgroups' and two of FP64 sums.
__host__ __device__ constexpr int64_t resident_all_words(int dt, int ldR, int grid) {
    return 2 * ((int64_t)grid * resident_words(dt, ldR) + 2 * ldR);
}

__device__ __forceinline__ void put_word(uint64_t *p, uint32_t v, uint32_t number) {
    __hip_atomic_store(p, (uint64_t)number << 32 | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t get_word(const uint64_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool has_number(uint64_t w, uint32_t number) { return (uint32_t)(w >> 32) == number; }
__device__ __forceinline__ double from_words(uint64_t lo, uint64_t hi) {
    return __hiloint2double((int)(uint32_t)hi, (int)(uint32_t)lo);
}

// The value in one word (FP32) or two (FP64).
template <int W>
__device__ __forceinline__ double value_of(const uint64_t (&u)[W]) {
    if constexpr (W == 2)
        return from_words(u[0], u[1]);
    else
        return (double)__uint_as_float((uint32_t)u[0]);
}

// The sum of column c over the workgroups [g0, g1), at most U of them, in
// order, FP64.  All words are requested together, slots past g1 reading the
// last one.
template <int DT, int U>
__device__ __forceinline__ bool sum_column(const uint64_t *set, int stride, int ldR, int c, int g0, int g1,
                                           uint32_t number, Ctrl *ctl, int64_t timeout_ticks, double *sum) {
    constexpr int W = DT == 0 ? 2 : 1;
    uint64_t u[U][W];
    WaitClock wait;
    for (;;) {
        bool all = true;
#pragma unroll
        for (int k = 0; k < U; ++k)
#pragma unroll
            for (int w = 0; w < W; ++w) u[k][w] = get_word(set + (int64_t)min(g0 + k, g1 - 1) * stride + w * ldR + c);
#pragma unroll
        for (int k = 0; k < U; ++k)
#pragma unroll
            for (int w = 0; w < W; ++w) all &= has_number(u[k][w], number);
        if (all) break;
        if (!wait.goes_on(ctl, timeout_ticks)) return false;
    }
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < U; ++k) {
        const double v = value_of(u[k]);
        s += g0 + k < g1 ? v : 0.0;
    }
    *sum = s;
    return true;
}

template <int DT>
__device__ __forceinline__ typename Store<DT>::Acc widen(typename Store<DT>::T v) {
    if constexpr (DT == 2)
        return __uint_as_float((uint32_t)v << 16);
    else
        return v;
}

constexpr int kResidentMaxCols = 512;   // LDS row length limit (8 columns per lane)
constexpr int kResidentMaxGrid = 32;    // workgroups of a resident launch at most
constexpr int kResidentThreads = 512;   // threads of a resident workgroup (8 wavefronts)
constexpr int kResidentWaves = kResidentThreads / 64;
constexpr int kSumSlots = kResidentThreads + kResidentMaxGrid;  // doubles of the exchange of sums
constexpr int kResidentRowsAtOnce = 4;  // rows a wavefront sweeps at once
constexpr int kResidentStaticLds = 1024; // bytes of static LDS a resident workgroup uses at most

// CPL = columns per lane (the LDS row length is 64 CPL); a template
// parameter, so that a row's loads are issued together and its values stay in
// registers between the dot products and the sum of positive slices.
template <int DT, int CPL>
__global__ __launch_bounds__(kResidentThreads) void resident_iterate(const ResidentArgs a) {
    using S = Store<DT>;
    using T = typename S::T;
    using Acc = typename S::Acc;
    constexpr int ldR = 64 * CPL;
    constexpr int NT = kResidentThreads, NW = kResidentWaves, RA = kResidentRowsAtOnce;
    constexpr int CPT = (ldR + NT - 1) / NT;   // columns per thread in the column-wise phases
    static_assert(NW * RA <= 64, "one wavefront reduces the rows' shares");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int G = (int)gridDim.x, g = (int)blockIdx.x;
    const int64_t r0 = (int64_t)g * a.rows;
    const int nr = (int)max((int64_t)0, min(a.m, r0 + a.rows) - r0);

    // LDS: the band of rows, its b, ||a_i||^2 and ||a_i||, the FP64 x, y
    // and translation sum, x and v in the accumulation type, the
    // wavefronts' partial y
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    auto up16 = [](size_t v) { return (v + 15) & ~(size_t)15; };
    size_t off = 0;
    T *As = reinterpret_cast<T *>(lds);
    off += up16((size_t)a.rows * ldR * sizeof(T));
    double *bs = reinterpret_cast<double *>(lds + off);
    off += up16((size_t)a.rows * sizeof(double));
    double *nus = reinterpret_cast<double *>(lds + off);
    off += up16((size_t)a.rows * sizeof(double));
    double *snus = reinterpret_cast<double *>(lds + off);
    off += up16((size_t)a.rows * sizeof(double));
    double *x64 = reinterpret_cast<double *>(lds + off);
    off += (size_t)ldR * sizeof(double);
    double *y64 = reinterpret_cast<double *>(lds + off);
    off += (size_t)ldR * sizeof(double);
    double *ws = reinterpret_cast<double *>(lds + off);
    off += (size_t)ldR * sizeof(double);
    Acc *xa = reinterpret_cast<Acc *>(lds + off);
    off += up16((size_t)ldR * sizeof(Acc));
    Acc *va = reinterpret_cast<Acc *>(lds + off);
    off += up16((size_t)ldR * sizeof(Acc));
    double *ysum = reinterpret_cast<double *>(lds + off);   // [SL][ldR] or [G][ldR / G]
    off += kSumSlots * sizeof(double);
    Acc *yw = reinterpret_cast<Acc *>(lds + off);   // [NW][ldR]
    __shared__ double hw[NW * RA], dw[NW * RA], bw[NW * RA], qw[NW];
    __shared__ State st_shared;   // the decision, taken by the last wavefront
    __shared__ int gave_up;
    static_assert((3 * NW * RA + NW) * sizeof(double) + sizeof(State) + sizeof(int) <= kResidentStaticLds,
                  "static LDS within what the host plans for");

    if (tid == 0) gave_up = 0;
    // the band, the committed state and the vectors
    const T *Ag = reinterpret_cast<const T *>(a.A);
    for (int i = tid; i < nr * ldR; i += NT) {
        const int r = i / ldR, c = i - r * ldR;
        As[i] = c < a.n ? Ag[(r0 + r) * a.ldA + c] : (T)0;
    }
    for (int i = tid; i < nr; i += NT) {
        bs[i] = a.b[r0 + i];
        nus[i] = a.nu[r0 + i];
        snus[i] = sqrt(nus[i]);
    }
    // every thread holds the state and takes every decision itself (the same
    // arithmetic on the same values in every thread of every workgroup);
    // the step limit and the schedule length do not change during a launch
    State st = load_global(&a.ctl->st[slot_of(a.j0 - 1)]);
    const int64_t step_limit = load_global(&a.ctl->step_limit);
    const int64_t sched_len = load_global(&a.ctl->sched_len);
    {
        const bool pv = st.vpend_valid != 0;
        const int64_t vi = st.v_idx;
        for (int c = tid; c < ldR; c += NT) {
            const bool in = c < a.n;
            const double xv = in ? a.x[c] : 0.0;
            const double vv = in ? (pv ? a.vpend[c] : 0.0) + ((a.V && vi >= 0) ? a.V[vi * a.ldV + c] : 0.0) : 0.0;
            x64[c] = xv;
            xa[c] = (Acc)xv;
            va[c] = (Acc)vv;
            ws[c] = in ? a.wsum[c] : 0.0;
            y64[c] = in ? a.y[c] : 0.0;
        }
    }
    __syncthreads();

    constexpr int WL = resident_words(DT, ldR);
    static_assert(CPT == 1, "a thread holds one column at most");
    constexpr int W = DT == 0 ? 2 : 1;
    // How the sums over the workgroups are formed: of up to eight by a thread
    // for each column; of more, rows of up to 128 columns by SL threads for
    // each, PER workgroups to a thread.  Longer rows take two trips: every
    // workgroup sums its share of the columns and passes the sums on.  Read by
    // all, G partials of FP64 rows of 256 are 128 KB a workgroup, and took
    // 5.9 us an iteration of 256 x 1024 for 4.9 in two trips (FP32 500 x 1400
    // 7.2 and 5.8; short rows lose by the second trip, FP64 64 x 128 3.7 and
    // 4.3, FP32 128 x 2000 4.3 and 5.0).
    constexpr int SL = 4, PER = kResidentMaxGrid / SL;
    const bool slices = CPL <= 2 && G > PER, two = CPL > 2 && G > PER;
    static_assert(CPL > 2 || SL * ldR <= NT, "a thread for each");
    bool failed = false;
    for (int64_t it = 0; it < a.K; ++it) {
        // the state this sweep runs under
        if (st.status != ST_RUNNING) break;
        const bool pv = st.vpend_valid != 0;
        const int64_t vi = st.v_idx, sp = st.sched_pos;
        const bool apply = pv || vi >= 0;
        const uint32_t number = a.base + (uint32_t)it;
        uint64_t *set = a.words + (it & 1) * (int64_t)kResidentMaxGrid * WL;
        uint64_t *mine = set + (int64_t)g * WL;
        Acc xr[CPL], vr[CPL], yacc[CPL];
#pragma unroll
        for (int k = 0; k < CPL; ++k) {
            xr[k] = xa[lane + 64 * k];
            vr[k] = apply ? va[lane + 64 * k] : (Acc)0;
            yacc[k] = (Acc)0;
        }
        // lane 16j of a wavefront settles row j of each of its batches and
        // keeps that row's share of h, dmax and ||b||inf
        static_assert(RA == 4, "the four rows of a batch are reduced together");
        const int jl = lane >> 4;
        const bool settler = (lane & 15) == 0;
        double h = 0.0, dmax = 0.0, binf = 0.0;
        // (compiled with and without the translation of the data)
        auto sweep_band = [&](auto with_translation) {
            constexpr bool AP = decltype(with_translation)::value;
            // wavefront w takes rows w, w + NW, w + 2 NW, ..., RA of them at a
            // time and without branches, so that their loads, dot products,
            // wavefront sums and divisions overlap (rows past the band count as
            // satisfied and are not written)
            for (int base = 0; base < nr; base += NW * RA) {
                Acc av[RA][CPL], dot[RA], tdot[RA];
                bool ok[RA];
#pragma unroll
                for (int j = 0; j < RA; ++j) {
                    const int r = base + wave + NW * j;
                    ok[j] = r < nr;
                    const T *row = As + (ok[j] ? r : 0) * ldR;
#pragma unroll
                    for (int k = 0; k < CPL; ++k) av[j][k] = widen<DT>(row[lane + 64 * k]);
                    dot[j] = (Acc)0;
                    tdot[j] = (Acc)0;
#pragma unroll
                    for (int k = 0; k < CPL; ++k) {
                        dot[j] = fma(xr[k], av[j][k], dot[j]);
                        if constexpr (AP) tdot[j] = fma(vr[k], av[j][k], tdot[j]);
                    }
                }
                const double dj = quad_total(dot[0], dot[1], dot[2], dot[3]);
                double tj = 0.0;
                if constexpr (AP) tj = quad_total(tdot[0], tdot[1], tdot[2], tdot[3]);
                const int rj = base + wave + NW * jl;
                const bool okj = settler && rj < nr;
                const int rc = okj ? rj : 0;
                double bb = bs[rc];
                if constexpr (AP) bb += tj;
                const double rr = okj ? dj - bb : -1.0;
                if (okj) {
                    bs[rj] = bb;
                    binf = max_nan(binf, fabs(bb));
                }
                const bool pos = rr > 0.0;
                h += pos ? 1.0 : 0.0;
                const double d = rr / snus[rc];
                dmax = pos ? max_nan(dmax, d) : (rr != rr ? rr : dmax);
                const Acc w = pos ? (Acc)(rr / nus[rc]) : (Acc)0;
#pragma unroll
                for (int j = 0; j < RA; ++j) {
                    const Acc wj = lane_value(w, 16 * j);
#pragma unroll
                    for (int k = 0; k < CPL; ++k) yacc[k] = fma(wj, av[j][k], yacc[k]);
                }
            }
        };
        if (apply)
            sweep_band(std::integral_constant<bool, true>{});
        else
            sweep_band(std::integral_constant<bool, false>{});
        // the wavefronts' partials, summed in wavefront order
#pragma unroll
        for (int k = 0; k < CPL; ++k) yw[wave * ldR + lane + 64 * k] = yacc[k];
        if (settler) {
            hw[wave * RA + jl] = h;
            dw[wave * RA + jl] = dmax;
            bw[wave * RA + jl] = binf;
        }
        __syncthreads();
        // the workgroup's partial y and totals
#pragma unroll
        for (int k = 0; k < CPT; ++k) {
            const int c = tid + NT * k;
            if (c < ldR) {
                Acc sum = yw[c];
#pragma unroll
                for (int w = 1; w < NW; ++w) sum += yw[w * ldR + c];
                if constexpr (DT == 0) {
                    put_word(mine + c, (uint32_t)__double2loint(sum), number);
                    put_word(mine + ldR + c, (uint32_t)__double2hiint(sum), number);
                } else {
                    put_word(mine + c, __float_as_uint(sum), number);
                }
            }
        }
        if (wave == NW - 1) {   // the workgroup's shares of h, dmax, ||b||inf
            const bool in = lane < NW * RA;
            const double hh = wave_total(in ? hw[lane] : 0.0);   // integers below 2^53: exact
            const double dd = wave_max_nan(in ? dw[lane] : 0.0);
            const double bm = wave_max_nan(in ? bw[lane] : 0.0);
            if (lane < kTotalWords) {
                const uint32_t v = lane == 0   ? (uint32_t)hh
                                   : lane == 1 ? (uint32_t)__double2loint(dd)
                                   : lane == 2 ? (uint32_t)__double2hiint(dd)
                                   : lane == 3 ? (uint32_t)__double2loint(bm)
                                               : (uint32_t)__double2hiint(bm);
                put_word(mine + (WL - kTotalWords) + lane, v, number);
            }
        }
        // Before the wait (they depend on the state this sweep ran under
        // only): the translation this sweep applied joins the FP64 sum, and the
        // drift row due after a step (row sched_pos: the decision either takes
        // it or none) is requested, so that it arrives during the wait.
        const bool next_due = a.V && sp < sched_len;
        double vcand[CPT];
#pragma unroll
        for (int k = 0; k < CPT; ++k) {
            const int c = tid + NT * k;
            vcand[k] = (c < a.n && next_due) ? a.V[sp * a.ldV + c] : 0.0;
            if (c < a.n && apply) ws[c] += (pv ? a.vpend[c] : 0.0) + ((a.V && vi >= 0) ? a.V[vi * a.ldV + c] : 0.0);
        }
        // every workgroup: y as the sum of the G partials in workgroup order,
        // FP64, and ||y||^2 in a fixed order, by the threads that hold a
        // column; the totals (an integer sum and two maxima, exact in any
        // order) and the decision by the last wavefront, once, shared through
        // LDS (lanes past G read slot G-1 and are masked out).
        const bool decider = wave == NW - 1;
        bool here = true;
        double hr = 0.0, dr = 0.0, br = 0.0, ys = 0.0;
        const int sl = tid / ldR, c0 = tid - sl * ldR;
        auto read_totals = [&]() {
            const uint64_t *tw = set + (int64_t)min(lane, G - 1) * WL + (WL - kTotalWords);
            uint64_t u[kTotalWords];
            WaitClock wait;
            for (;;) {
                bool all = true;
#pragma unroll
                for (int k = 0; k < kTotalWords; ++k) u[k] = get_word(tw + k);
#pragma unroll
                for (int k = 0; k < kTotalWords; ++k) all &= has_number(u[k], number);
                if (all) break;
                if (!wait.goes_on(a.ctl, a.timeout_ticks)) return false;
            }
            hr = (double)(uint32_t)u[0];
            dr = from_words(u[1], u[2]);
            br = from_words(u[3], u[4]);
            return true;
        };
        if (two) {
            // the columns of this workgroup: everyone's partials, one or two to a thread
            const int B = (ldR + G - 1) / G, first = g * B;
            uint64_t u[2][W];
            WaitClock wait;
            for (;;) {
                bool all = true;
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const int i = min(tid + k * NT, G * B - 1), gg = i / B, c = min(first + i - gg * B, ldR - 1);
#pragma unroll
                    for (int w = 0; w < W; ++w) u[k][w] = get_word(set + (int64_t)gg * WL + w * ldR + c);
                }
#pragma unroll
                for (int k = 0; k < 2; ++k)
#pragma unroll
                    for (int w = 0; w < W; ++w) all &= has_number(u[k][w], number);
                if (all) break;
                if (!wait.goes_on(a.ctl, a.timeout_ticks)) {
                    here = false;
                    break;
                }
            }
#pragma unroll
            for (int k = 0; k < 2; ++k)
                if (tid + k * NT < G * B) ysum[tid + k * NT] = value_of(u[k]);
            if (!here) gave_up = 1;
            __syncthreads();
            uint64_t *sums = a.words + 2 * (int64_t)kResidentMaxGrid * WL + (it & 1) * (int64_t)(2 * ldR);
            if (tid < B && first + tid < ldR && !gave_up) {
                double s = 0.0;
                for (int gg = 0; gg < G; ++gg) s += ysum[gg * B + tid];
                put_word(sums + first + tid, (uint32_t)__double2loint(s), number);
                put_word(sums + ldR + first + tid, (uint32_t)__double2hiint(s), number);
            }
            if (decider) here = read_totals() && here;
            if (tid < ldR)
                here = sum_column<0, 1>(sums, 0, ldR, tid, 0, 1, number, a.ctl, a.timeout_ticks, &ys) && here;
        } else {
            const int g0 = slices ? sl * PER : 0, g1 = min(G, g0 + PER);
            if (sl < (slices ? SL : 1) && g0 < g1)
                here = sum_column<DT, PER>(set, WL, ldR, c0, g0, g1, number, a.ctl, a.timeout_ticks, &ys);
            if (slices && sl < SL) ysum[sl * ldR + c0] = ys;
            if (decider) here = read_totals() && here;
        }
        if (!here) gave_up = 1;
        if (slices) {
            __syncthreads();
            ys = 0.0;
            if (tid < ldR)
#pragma unroll
                for (int k = 0; k < SL; ++k) ys += ysum[k * ldR + tid];
        }
        double q = 0.0;
        if (tid < ldR) {
            y64[tid] = ys;
            q = ys * ys;
        }
        if (wave * 64 < ldR) q = wave_total(q);   // (the other wavefronts hold no column)
        if (lane == 0) qw[wave] = q;
        Totals t{};
        if (decider) {   // (while the other wavefronts wait for their loads)
            t.h = (int64_t)wave_total(lane < G ? hr : 0.0);   // integers below 2^53: exact
            t.dmax = wave_max_nan(lane < G ? dr : 0.0);
            t.binf = wave_max_nan(lane < G ? br : 0.0);
        }
        __syncthreads();
        if (gave_up) {
            failed = true;
            break;
        }
        if (decider) {
            double qq = qw[0];
#pragma unroll
            for (int w = 1; w < NW; ++w) qq += qw[w];
            const State s = decide(st, t, sqrt(qq), a.dp, step_limit, sched_len);
            if (lane == 0) st_shared = s;
        }
        __syncthreads();
        st = st_shared;
        // the step (x <- x - s y, one rounding) and the translation due at the
        // next sweep (the row requested before the wait, when one is due)
        const double step = st.s;
        const bool take = st.v_idx >= 0;
#pragma unroll
        for (int k = 0; k < CPT; ++k) {
            const int c = tid + NT * k;
            if (c >= a.n) continue;
            if (step != 0.0) x64[c] = step_point(x64[c], step, y64[c]);
            xa[c] = (Acc)x64[c];
            va[c] = take ? (Acc)vcand[k] : (Acc)0;
        }
        __syncthreads();
    }
    if (failed) {
        if (g == 0 && tid == 0 && a.progress) post_progress(a.progress, a.j0 + a.K - 1, ST_FAULT);
        return;
    }

    // write back: the band's b; workgroup 0 the vectors and the state
    for (int i = tid; i < nr; i += NT) a.b[r0 + i] = bs[i];
    if (g != 0) return;
    const State p = st;
    const double *vrow_next = (a.V && p.v_idx >= 0) ? a.V + p.v_idx * a.ldV : nullptr;
    Acc *wx = reinterpret_cast<Acc *>(a.work);
    for (int c = tid; c < a.n; c += NT) {
        a.x[c] = x64[c];
        a.y[c] = y64[c];
        a.wsum[c] = ws[c];
        wx[c] = (Acc)x64[c];
        wx[a.ldA + c] = vrow_next ? (Acc)vrow_next[c] : (Acc)0;
        wx[2 * a.ldA + c] = (Acc)y64[c];
    }
    if (tid == 0) {
        store_global(&a.ctl->st[0], p);
        store_global(&a.ctl->st[1], p);
        if (a.progress) post_progress(a.progress, a.j0 + a.K - 1, p.status);
    }
}

}  // namespace modap
