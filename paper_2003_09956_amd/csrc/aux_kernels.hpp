// Kernels around the sweep: row norms, the fixed-order reduction of the
// partial y, the stage kernel that settles each iteration, control-block
// updates made between calls, in-place row replacement and the exact
// right-hand side read back by a query.
#pragma once

#include "modap_device.hpp"
#include "readback.hpp"

namespace modap {

template <int DT>
__device__ __forceinline__ double load_elem(const void *A, int64_t idx) {
    if constexpr (DT == 0) {
        return reinterpret_cast<const double *>(A)[idx];
    } else if constexpr (DT == 1) {
        return (double)reinterpret_cast<const float *>(A)[idx];
    } else {
        const uint32_t u = ((uint32_t)reinterpret_cast<const uint16_t *>(A)[idx]) << 16;
        return (double)__uint_as_float(u);
    }
}

// One 16-byte vector of a row in FP64 (exact).
template <int DT>
__device__ __forceinline__ void unpack64(const uint4 u, double (&v)[Store<DT>::VEC]) {
    if constexpr (DT == 0) {
        v[0] = __hiloint2double((int)u.y, (int)u.x);
        v[1] = __hiloint2double((int)u.w, (int)u.z);
    } else {
        const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if constexpr (DT == 1) {
                v[k] = (double)__uint_as_float(w[k]);
            } else {
                v[2 * k] = (double)__uint_as_float(w[k] << 16);
                v[2 * k + 1] = (double)__uint_as_float(w[k] & 0xffff0000u);
            }
        }
    }
}
template <int DT>
__device__ __forceinline__ void load_vec64(const void *A, int64_t idx, double (&v)[Store<DT>::VEC]) {
    unpack64<DT>(*reinterpret_cast<const uint4 *>(reinterpret_cast<const typename Store<DT>::T *>(A) + idx), v);
}

template <int N>
__device__ __forceinline__ void load_f64(const double *p, double (&v)[N]) {
    static_assert(N % 2 == 0, "whole 16-byte vectors");
#pragma unroll
    for (int e = 0; e < N; e += 2) {
        const double2 t = *reinterpret_cast<const double2 *>(p + e);
        v[e] = t.x;
        v[e + 1] = t.y;
    }
}

// Rows that a wavefront of the FP64 passes over A takes together: the vectors
// the rows are multiplied with (8 bytes an element, where BF16 rows have 2)
// are then read from L1 once for four rows, which keeps the passes bound by
// HBM.  With one row per wavefront and one element per load, the certificate's
// pass over 128 MiB of BF16 rows took 104 us and rhs_exact's 55 us.
constexpr int kRows64 = 4;

// nu_i = ||a_i||^2 in FP64 (section 2: the denominator of the reflection
// vector).  One wavefront per row, a fixed summation order, 16-byte loads, four
// in flight.  Bound by the read of A.  (With one element a load, one after
// another, set_system of 2.1 GB of BF16 rows took 2.5 ms, now 1.7; the norms of
// 777 x 3000 FP64 7.1 us, now 3.9 with x staged beside them.)  Reports the
// first zero or non-finite row
// through *bad (atomic minimum of the index).
template <int DT>
__device__ __forceinline__ void row_norm(const void *A, int64_t ldA, int64_t m, int64_t n, double *nu,
                                         unsigned long long *bad, int64_t block) {
    constexpr int VEC = Store<DT>::VEC, U = 4;
    const int lane = threadIdx.x & 63;
    const int64_t row = block * 4 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (row >= m) return;
    const int64_t bytes = ldA * (int64_t)sizeof(typename Store<DT>::T);
    const char *p = reinterpret_cast<const char *>(A) + row * bytes;
    double s = 0.0;
    for (int64_t c = 0; c * 1024 < bytes; c += U) {
        uint4 u[U];
#pragma unroll
        for (int k = 0; k < U; ++k)
            u[k] = load_cached_vec(window_resource(p, bytes, (c + k) * 1024, 1024), (uint32_t)(lane * 16));
#pragma unroll
        for (int k = 0; k < U; ++k) {
            double e[VEC];
            unpack64<DT>(u[k], e);
            const int64_t col = ((c + k) * 64 + lane) * VEC;
#pragma unroll
            for (int q = 0; q < VEC; ++q) {
                const double v = col + q < n ? e[q] : 0.0;   // (a caller's rows may hold anything past n)
                s = __fma_rn(v, v, s);
            }
        }
    }
    s = wave_total(s);
    if (lane == 0) {
        nu[row] = s;
        if (!(s > 0.0) || !isfinite(s)) atomicMin(bad, (unsigned long long)row);
    }
}
template <int DT>
__global__ __launch_bounds__(256) void row_norms(const void *A, int64_t ldA, int64_t m, int64_t n, double *nu,
                                                 unsigned long long *bad) {
    row_norm<DT>(A, ldA, m, n, nu, bad, blockIdx.x);
}

// Raises *flag when any of p[0..np) or q[0..nq) is NaN or infinite.
__global__ void check_finite(const double *p, int64_t np, const double *q, int64_t nq, unsigned long long *flag) {
    const int64_t first = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    bool bad = false;
    for (int64_t i = first; i < np; i += step) bad |= !isfinite(p[i]);
    for (int64_t i = first; i < nq; i += step) bad |= !isfinite(q[i]);
    if (bad) atomicOr(flag, 1ull);
}

// Threads of a reduction workgroup.  Measured on the FP32 n = 8192 system
// with 256 partials: 256 threads took 5.2 us, 1024 threads 6.9 us (with
// permute-unit sums and 8 loads in flight; 4.3 us now at 256).
constexpr int kReduceThreads = 256;

// Column sums of the workgroup partials of y, in a fixed order, in FP64.
// Workgroup b writes its share of ||y||^2 to ynp[b]; workgroup 0 also forms
// the totals of h, dmax and binf.  The stop test and the step are taken from
// these by the next sweep (or by the stage kernel at the end of a call).  In
// iteration mode it first makes the previous step permanent in x and then
// writes the working vectors of the next sweep.
template <typename Acc>
__global__ __launch_bounds__(kReduceThreads) void reduce_y(const ReduceArgs a) {
    constexpr int COLS = 64;                    // columns per workgroup
    constexpr int VW = 16 / (int)sizeof(Acc);   // columns per 16-byte load
    constexpr int LPRR = COLS / VW;             // lanes per partial row
    constexpr int RPW = 64 / LPRR;              // partial rows per wavefront load
    constexpr int NWR = kReduceThreads / 64;    // wavefronts per workgroup
    constexpr int RG = NWR * RPW;               // row groups per workgroup
    constexpr int U = 16;                       // loads in flight per lane
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wv = tid >> 6;
    const int rg = (tid >> 6) * RPW + lane / LPRR;
    const int cl = lane % LPRR;
    const int64_t col = (int64_t)blockIdx.x * COLS + tid;   // column of threads 0..63
    // ldPart is a multiple of 64 and covers every workgroup's columns
    const Acc *pc = reinterpret_cast<const Acc *>(a.part) + (int64_t)blockIdx.x * COLS + cl * VW;

    // Every load that does not depend on the state is issued before the state
    // is examined: the first batch of partial rows, the column's x and
    // previous y, and (workgroup 0) the first scalar partials.
    uint4 v[U];
    auto issue = [&](int g0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int g = min(g0 + u * RG, a.G - 1);
            v[u] = *reinterpret_cast<const uint4 *>(pc + (int64_t)g * a.ldPart);
        }
    };
    issue(rg);
    const bool colw = a.work && tid < COLS && col < a.n;
    double xo = 0.0, yo = 0.0, wso = 0.0;
    int64_t slen = 0;
    if (colw) {
        xo = load_global(a.x + col);
        yo = load_global(a.y + col);
        if (a.wsum) wso = load_global(a.wsum + col);
        if (a.V) slen = load_global(&a.ctl->sched_len);
    }
    int64_t h = 0;
    double dm = 0.0, bm = 0.0;
    if (blockIdx.x == 0 && tid < a.Gs) {
        h = load_global(a.h_part + tid);
        dm = load_global(a.dmax_part + tid);
        bm = load_global(a.binf_part + tid);
    }
    State S{};
    if (a.iterate) {
        S = load_global(&a.ctl->st[slot_of(a.j - 1)]);
        if (S.status != ST_RUNNING) return;
    }
    // The drift row due next depends on the state only: requested now, so
    // that it arrives while the partial rows are summed.  So is the
    // translation this sweep applied (one-shot part and drift row), which is
    // added to the running sum of translations in FP64.
    const bool due = colw && a.V && S.sched_pos < slen;
    const double vdue = due ? load_global(a.V + S.sched_pos * a.ldV + col) : 0.0;
    const bool ap = colw && a.wsum && a.has_v && S.vpend_valid;
    const bool ar = colw && a.wsum && a.has_v && a.V && S.v_idx >= 0;
    const double vap = (ap ? load_global(a.vpend + col) : 0.0) + (ar ? load_global(a.V + S.v_idx * a.ldV + col) : 0.0);

    // Batches of U independent 16-byte loads (partial rows rg, rg+RG, ...),
    // each batch summed in order, batches in order: a fixed order for a given G.
    double acc[VW];
#pragma unroll
    for (int k = 0; k < VW; ++k) acc[k] = 0.0;
    for (int g0 = rg; g0 < a.G; g0 += U * RG) {
        if (g0 != rg) issue(g0);
#pragma unroll
        for (int k = 0; k < VW; ++k) {
            double bsum = 0.0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                Acc e[VW];
                __builtin_memcpy(e, &v[u], 16);
                if (g0 + u * RG < a.G) bsum += (double)e[k];
            }
            acc[k] += bsum;
        }
    }
    __shared__ double sh[RG][COLS];
#pragma unroll
    for (int k = 0; k < VW; ++k) sh[rg][cl * VW + k] = acc[k];
    __syncthreads();
    if (tid < 64) {
        double yv = 0.0;
#pragma unroll 8
        for (int r = 0; r < RG; ++r) yv += sh[r][tid];
        double sq = 0.0;
        if (col < a.n) {
            if (colw) {
                // the step decided on the previous check becomes permanent in
                // FP64, then the working vectors of the next sweep: x, the
                // drift row due next (applied if the next decision moves on),
                // and this sweep's y
                if (a.apply_step && S.s != 0.0) {
                    xo = step_point(xo, S.s, yo);
                    a.x[col] = xo;
                }
                Acc *w = reinterpret_cast<Acc *>(a.work);
                w[col] = (Acc)xo;
                w[a.ldA + col] = (Acc)vdue;
                w[2 * a.ldA + col] = (Acc)yv;
                if (ap || ar) a.wsum[col] = wso + vap;
            }
            a.y[col] = yv;
            sq = yv * yv;
        }
        sq = wave_total(sq);
        if (tid == 0) a.ynp[blockIdx.x] = sq;
    }
    if (blockIdx.x != 0) {
        if (a.view) announce(a.view, a.arrived, a.seq, gridDim.x);
        return;
    }

    for (int g = tid + kReduceThreads; g < a.Gs; g += kReduceThreads) {
        h += a.h_part[g];
        dm = max_nan(dm, a.dmax_part[g]);
        bm = max_nan(bm, a.binf_part[g]);
    }
    // across each wavefront with DPP moves (no permute round trips): h as an
    // FP64 sum of integers below 2^53 (exact), the maxima in any order
    h = (int64_t)wave_total((double)h);
    dm = wave_max_nan(dm);
    bm = wave_max_nan(bm);
    __shared__ int64_t hw[NWR];
    __shared__ double dw[NWR], bw[NWR];
    if (lane == 0) {
        hw[wv] = h;
        dw[wv] = dm;
        bw[wv] = bm;
    }
    __syncthreads();
    if (tid == 0) {
        Totals t{};
        for (int w = 0; w < NWR; ++w) {
            t.h += hw[w];
            t.dmax = max_nan(t.dmax, dw[w]);
            t.binf = max_nan(t.binf, bw[w]);
        }
        *a.tot = t;
        if (a.h_out) *a.h_out = t.h;
        if (a.dmax_out) *a.dmax_out = t.dmax;
        if (a.view) {
            a.view->tot = t;
            a.view->fault = *a.fault;
        }
    }
    if (a.view) announce(a.view, a.arrived, a.seq, gridDim.x);
}

// End of a call: settle the last check j (no sweep follows to do it).  Every
// workgroup takes the decision from the check's totals (the same arithmetic in
// every workgroup), workgroup 0 records it in slot j & 1, and each workgroup,
// for its columns, makes the step permanent in FP64 (x <- x - s*y, eq. 12 or
// Algorithm 1) and writes x and the translation due next into the working
// vectors.
template <typename Acc>
__global__ __launch_bounds__(256) void stage_iter(const StageArgs a) {
    const State p = a.ctl->st[slot_of(a.j - 1)];
    if (p.status != ST_RUNNING) {
        if (blockIdx.x == 0 && threadIdx.x == 0) a.ctl->st[slot_of(a.j)] = p;
        return;
    }
    __shared__ State sst;
    if (threadIdx.x < 64) {
        const double yn = ynorm_of(a.ynp, a.R, threadIdx.x);
        const State cur = decide(p, *a.tot, yn, a.dp, a.ctl->step_limit, a.ctl->sched_len);
        if (threadIdx.x == 0) {
            sst = cur;
            if (blockIdx.x == 0) a.ctl->st[slot_of(a.j)] = cur;
        }
    }
    __syncthreads();
    const double s = sst.s;
    const double *vrow = (a.V && sst.v_idx >= 0) ? a.V + sst.v_idx * a.ldV : nullptr;
    Acc *wx = reinterpret_cast<Acc *>(a.work);
    Acc *wv = wx + a.ldA;
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < a.n;
         j += (int64_t)gridDim.x * blockDim.x) {
        double xv = a.x[j];
        if (s != 0.0) {
            xv = step_point(xv, s, a.y[j]);
            a.x[j] = xv;
        }
        wx[j] = (Acc)xv;
        wv[j] = vrow ? (Acc)vrow[j] : (Acc)0;
    }
}

// Working vectors for the first sweep of a call (or an evaluation) from the
// committed state in slot (j-1)&1: x as it is, and the pending translation
// (one-shot part plus the drift row due).
template <typename Acc>
__global__ __launch_bounds__(256) void prime_work(const StageArgs a) {
    const State &p = a.ctl->st[slot_of(a.j - 1)];
    const bool use_p = p.vpend_valid != 0;
    const double *vrow = (a.V && p.v_idx >= 0) ? a.V + p.v_idx * a.ldV : nullptr;
    Acc *wx = reinterpret_cast<Acc *>(a.work);
    Acc *wv = wx + a.ldA;
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < a.n;
         j += (int64_t)gridDim.x * blockDim.x) {
        const double v = (use_p ? a.vpend[j] : 0.0) + (vrow ? vrow[j] : 0.0);
        wx[j] = (Acc)a.x[j];
        wv[j] = (Acc)v;
    }
}

// The control kernels below run between calls as a single thread (or a
// single workgroup) on the committed state in slot `sl`.

// Start of an iterate/solve call: a stop that came from a previous call's
// tolerance, step limit or missing direction is re-examined by the next sweep.
__global__ void ctl_begin(Ctrl *c, int sl, int64_t max_steps) {
    if (threadIdx.x != 0) return;
    State &s = c->st[sl];
    if (s.status == ST_CONVERGED || s.status == ST_LIMIT || s.status == ST_NO_DIRECTION) s.status = ST_RUNNING;
    c->step_limit = max_steps < 0 ? INT64_MAX : s.steps + max_steps;
}

// A fresh state (set_system): both slots.
__device__ __forceinline__ void fresh_state(Ctrl *c) {
    State s{};
    s.v_idx = -1;
    s.status = ST_RUNNING;
    c->st[0] = s;
    c->st[1] = s;
    c->step_limit = INT64_MAX;
    c->sched_len = 0;
    c->fault = 0;
}

__global__ void ctl_init(Ctrl *c, DataChecks *checks) {
    if (threadIdx.x != 0) return;
    *checks = DataChecks{ULLONG_MAX, 0};
    fresh_state(c);
}

// All that a stateless sweep of a caller's arrays needs first, in one launch:
// the row norms (workgroups below `norms`), x in the accumulation type with
// the rest of the working vectors zero, and a fresh state to run under.
template <int DT>
__global__ __launch_bounds__(256) void static_begin(const void *A, int64_t ldA, int64_t m, int64_t n, double *nu,
                                                    unsigned long long *bad, const double *x, void *work, Ctrl *ctl,
                                                    int norms) {
    using Acc = typename Store<DT>::Acc;
    if ((int)blockIdx.x < norms) {
        row_norm<DT>(A, ldA, m, n, nu, bad, blockIdx.x);
        return;
    }
    const int64_t first = (int64_t)((int)blockIdx.x - norms) * 256 + threadIdx.x;
    if (first == 0) fresh_state(ctl);
    Acc *w = reinterpret_cast<Acc *>(work);
    for (int64_t j = first; j < ldA; j += (int64_t)((int)gridDim.x - norms) * 256) {
        w[j] = j < n ? (Acc)x[j] : (Acc)0;
        w[ldA + j] = (Acc)0;
        w[2 * ldA + j] = (Acc)0;
    }
}

// A new approximation: counters restart, no step is pending.
__global__ void ctl_restart(Ctrl *c, int sl) {
    if (threadIdx.x != 0) return;
    State &s = c->st[sl];
    if (s.status != ST_BAD_ROW) s.status = ST_RUNNING;
    s.s = 0.0;
    s.steps = 0;
    s.sweeps = 0;
    s.dmax = s.binf = s.ynorm = s.eps_abs = 0.0;
    s.h = 0;
    s.feasible = 0;
}

// One-shot translation: vpend <- (pending ? vpend : 0) + v.  A single
// workgroup, so the pending flag is read before it is set.
__global__ __launch_bounds__(1024) void vpend_add(Ctrl *c, int sl, double *vpend, const double *v, int64_t n) {
    const int valid = c->st[sl].vpend_valid;
    for (int64_t j = threadIdx.x; j < n; j += blockDim.x) vpend[j] = valid ? vpend[j] + v[j] : v[j];
    __syncthreads();
    if (threadIdx.x == 0) c->st[sl].vpend_valid = 1;
}

// Move a drift-schedule translation that is due at the next sweep into the
// one-shot slot (used before the schedule buffer is replaced or b is read).
__global__ __launch_bounds__(1024) void sched_to_vpend(Ctrl *c, int sl, double *vpend, const double *V,
                                                       int64_t ldV, int64_t n) {
    const int64_t idx = c->st[sl].v_idx;
    const int valid = c->st[sl].vpend_valid;
    if (idx >= 0 && V) {
        for (int64_t j = threadIdx.x; j < n; j += blockDim.x)
            vpend[j] = (valid ? vpend[j] : 0.0) + V[idx * ldV + j];
    }
    __syncthreads();
    if (threadIdx.x == 0 && idx >= 0) {
        c->st[sl].vpend_valid = V ? 1 : valid;
        c->st[sl].v_idx = -1;
    }
}

__global__ void clear_words(uint64_t *p, int64_t count) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x) p[i] = 0;
}

__device__ __forceinline__ void start_schedule(Ctrl *c, int sl, int64_t T) {
    c->sched_len = T;
    c->st[sl].sched_pos = 0;
    c->st[sl].v_idx = -1;
}

__global__ void ctl_set_drift(Ctrl *c, int sl, int64_t T) {
    if (threadIdx.x == 0) start_schedule(c, sl, T);
}

// A drift schedule in device memory taken in with one pass: T rows of n at
// stride ldv copied to rows of ldA (zeros past n) and checked; the last
// workgroup starts the schedule, or one of no rows if an entry is not finite,
// and tells the host which.  (Cleared, copied by a copy engine, checked and
// the flag copied back, behind a free, an allocation and two waits, a schedule
// of 16 rows of 1000 took 106 us; with this and a kept buffer 17.)  *flag and
// *arrived are zero between launches.  At most kDriftGroups workgroups: each
// arrival costs a release to the device (512 of them took 50 us).
constexpr int kDriftCols = 1024;
constexpr int kDriftGroups = 128;
__global__ __launch_bounds__(256) void drift_in(const double *src, int64_t ldv, int64_t n, int64_t T, double *V,
                                                int64_t ldA, unsigned long long *flag, Ctrl *ctl, int sl,
                                                HostView *view, uint32_t *arrived, uint32_t seq) {
    bool bad = false;
    const int64_t chunks = (ldA + kDriftCols - 1) / kDriftCols;   // a workgroup takes one chunk of a row at a time
    for (int64_t w = blockIdx.x; w < T * chunks; w += gridDim.x) {
        const int64_t row = w / chunks, col0 = w % chunks * kDriftCols + threadIdx.x;
        double v[kDriftCols / 256];
#pragma unroll
        for (int k = 0; k < kDriftCols / 256; ++k) {
            const int64_t col = col0 + k * 256;
            v[k] = col < n ? src[row * ldv + col] : 0.0;
        }
#pragma unroll
        for (int k = 0; k < kDriftCols / 256; ++k) {
            const int64_t col = col0 + k * 256;
            bad |= !isfinite(v[k]);
            if (col < ldA) V[row * ldA + col] = v[k];
        }
    }
    if (bad) atomicOr(flag, 1ull);
    __threadfence();
    __syncthreads();
    if (threadIdx.x != 0) return;
    if (gridDim.x > 1 &&
        __hip_atomic_fetch_add(arrived, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) != gridDim.x - 1)
        return;
    __hip_atomic_store(arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long any = atomicExch(flag, 0ull);
    start_schedule(ctl, sl, any ? 0 : T);
    view->fault = any != 0;
    __hip_atomic_store(&view->seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Row replacement in place (one workgroup per replaced row): copy the new
// coefficients, refresh ||a_i||^2, and store the right-hand sides.  A
// translation still pending for the next sweep (the one-shot part and the
// drift row due) has already happened to the data the caller sees, so it must
// not move the new row: b_i is stored as new_b - <a_new, pending>, which the
// next sweep's translation brings back to new_b.  The exact data are
// bref + A wsum, so bref_i = new_b - <a_new, wsum + pending>.  Nothing is
// written once the state holds ST_BAD_ROW (for instance after a duplicate
// device-side row index).
template <int DT>
__global__ __launch_bounds__(256) void scatter_rows(void *A, int64_t ldA, int64_t m, int64_t n,
                                                    const int64_t *rows, const void *new_rows,
                                                    const double *new_b, double *b, double *bref, double *nu,
                                                    Ctrl *ctl, int sl, const double *vpend, const double *V,
                                                    int64_t ldV, const double *wsum) {
    using T = typename Store<DT>::T;
    const int64_t q = blockIdx.x;
    const State st = load_global(&ctl->st[sl]);
    if (st.status == ST_BAD_ROW) return;
    const int64_t i = rows[q];
    if (i < 0 || i >= m) {
        if (threadIdx.x == 0) ctl->st[sl].status = ST_BAD_ROW;
        return;
    }
    const bool valid = st.vpend_valid != 0;
    const double *vrow = (V && st.v_idx >= 0) ? V + st.v_idx * ldV : nullptr;
    T *dst = reinterpret_cast<T *>(A) + i * ldA;
    const T *src = reinterpret_cast<const T *>(new_rows) + q * n;
    double s2 = 0.0, sv = 0.0, sw = 0.0;
    for (int64_t j = threadIdx.x; j < n; j += 256) {
        const T raw = src[j];
        dst[j] = raw;
        const double v = load_elem<DT>(src, j);
        s2 = __fma_rn(v, v, s2);
        const double pj = (valid ? vpend[j] : 0.0) + (vrow ? vrow[j] : 0.0);
        sv = __fma_rn(v, pj, sv);
        sw = __fma_rn(v, wsum[j], sw);
    }
    s2 = wave_sum(s2);
    sv = wave_sum(sv);
    sw = wave_sum(sw);
    __shared__ double p2[4], pv[4], pw[4];
    if ((threadIdx.x & 63) == 0) {
        p2[threadIdx.x >> 6] = s2;
        pv[threadIdx.x >> 6] = sv;
        pw[threadIdx.x >> 6] = sw;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const double t2 = ((p2[0] + p2[1]) + p2[2]) + p2[3];
        const double tv = ((pv[0] + pv[1]) + pv[2]) + pv[3];
        const double tw = ((pw[0] + pw[1]) + pw[2]) + pw[3];
        nu[i] = t2;
        b[i] = new_b[q] - tv;
        bref[i] = new_b[q] - (tw + tv);
        if (!(t2 > 0.0) || !isfinite(t2) || !isfinite(new_b[q])) ctl->st[sl].status = ST_BAD_ROW;
    }
}

// Device-side row indices of a replacement: one thread per index claims its
// row in `claim` (zero outside this pair of kernels); an index out of range or
// claimed twice puts the state in ST_BAD_ROW before any row is written.
__global__ void claim_rows(const int64_t *rows, int64_t k, int64_t m, int *claim, Ctrl *ctl, int sl) {
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < k; q += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = rows[q];
        if (i < 0 || i >= m || atomicAdd(claim + i, 1) != 0) ctl->st[sl].status = ST_BAD_ROW;
    }
}

// Releases the claims of claim_rows (after the replacement).
__global__ void release_rows(const int64_t *rows, int64_t k, int64_t m, int *claim) {
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < k; q += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = rows[q];
        if (i >= 0 && i < m) claim[i] = 0;
    }
}

// The right-hand side of the data as the caller sees them, in FP64 and
// without changing any state: out_i = bref_i + <a_i, wsum + pending>, with
// the pending translation (one-shot part and due drift row) of slot sl.
// kRows64 rows per wavefront, a fixed summation order; the vectors are padded
// with zeros to ldA (a multiple of 16 bytes), so whole 16-byte vectors of A
// are read.  Bound by the read of A: 128 MiB of BF16 rows in 55 us before, see
// kRows64.
template <int DT>
__global__ __launch_bounds__(256) void rhs_exact(const void *A, int64_t ldA, int64_t m, int64_t n, const Ctrl *ctl,
                                                 int sl, const double *bref, const double *wsum,
                                                 const double *vpend, const double *V, int64_t ldV, double *out) {
    constexpr int VEC = Store<DT>::VEC, R = kRows64;
    const State st = load_global(&ctl->st[sl]);
    const bool valid = st.vpend_valid != 0;
    const double *vrow = (V && st.v_idx >= 0) ? V + st.v_idx * ldV : nullptr;
    const int lane = threadIdx.x & 63;
    const int64_t row0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * R;
    if (row0 >= m) return;
    double s[R] = {};
#pragma unroll 2
    for (int64_t j = (int64_t)lane * VEC; j < ldA; j += 64 * VEC) {
        double t[VEC], e[R][VEC];
#pragma unroll
        for (int r = 0; r < R; ++r) load_vec64<DT>(A, min(row0 + r, m - 1) * ldA + j, e[r]);
        load_f64(wsum + j, t);
        if (valid || vrow) {
            double u[VEC] = {}, v[VEC] = {};
            if (valid) load_f64(vpend + j, u);
            if (vrow) load_f64(vrow + j, v);
#pragma unroll
            for (int k = 0; k < VEC; ++k) t[k] += u[k] + v[k];
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int k = 0; k < VEC; ++k) s[r] = __fma_rn(e[r][k], t[k], s[r]);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        s[r] = wave_total(s[r]);
        if (lane == 0 && row0 + r < m) out[row0 + r] = bref[row0 + r] + s[r];
    }
}

}  // namespace modap
