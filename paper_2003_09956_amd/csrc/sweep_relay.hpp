// One-read sweep for rows too long for one workgroup.
//
// The same sweep as sweep_wide.hpp (section 3's Map of positive slices and
// Reduce(+), the eq. 10 measures and the translation update) for rows longer
// than a workgroup's registers.  The row is cut into column tiles of equal
// width, the rows into bands, and each workgroup owns one (band, tile).  A
// row's weight needs the dot products of all its tiles, so the workgroups of a
// band pass their partial dots to each other while the rows wait on chip:
//
//   iteration t, streaming wavefronts: y += w(t-D) a(t-D) from LDS; the dot
//       products of row t, which is in registers; row t to LDS in the place of
//       row t-D; row t+P requested.
//   iteration t, publishing wavefront: makes the tile's dots of row t-1 known
//       (tile 0: the row's b too, when a translation may apply).
//   iteration t, weighing wavefront: requests every tile's dots of row
//       t-D+1+F, and from those of row t-D+1, requested F iterations ago,
//       forms w(t-D+1) = r/||a||^2 for the streaming wavefronts' next iteration.
//
// One barrier per iteration; A is read once, where the two-phase form
// (sweep_split.hpp) reads the violated rows again.  Bound by the read of A:
// FP64 box-plus-sum rows of n = 32000 (16.4 GB, half of them violated) took
// 3.81 ms an iteration in two phases and take 2.39 here (6.85 TB/s).
//
// The exchange has wavefronts of its own because a wait for its loads would
// otherwise be a wait for the rows in flight too (vector loads return in
// order).  D rows of LDS are the time it has: 128 KiB are about 4.7 us of a
// CU's share of HBM.  A published word takes about 1 us to where every XCD
// reads it and as long again to a peer's registers.
//
// Exchange: a partial dot travels as two 64-bit words, each half of its bits
// with a 32-bit number of the row that no other row of this launch or an
// earlier one left in the same place.  A word is therefore complete in itself:
// single-copy atomic at agent scope, no ordering between words is needed, no
// fence.  A workgroup publishes row r only after it has consumed row r+1-D of
// every peer; a peer that published that row may still have rows down to
// r+3-2D to read, so kRelayRing slots >= 2D-2 never overwrite an unread word.
//
// b is translated in place, so nobody reads it while another workgroup may
// write it: tile 0 alone reads and writes it, and passes it on with its dots
// (two more words of a row).  Its publishing wavefront holds the b of 64 rows
// at a time, in registers by the time the first of them, row 64 q, is
// published in iteration 64 q + 1; its weighing wavefront, D-3 or more barriers
// later, is the only one to write them.  (With b read by every tile, a peer up
// to D-2 iterations behind could read rows that tile 0 had translated already
// and add the translation twice.)  A launch that cannot translate writes no b,
// and every tile reads it.
//
// The launch is cooperative (every workgroup resident).  A wait is bounded by
// the constant clock as in resident.hpp: a workgroup that has waited too long
// raises ctl->fault, waits no more and goes through the rest of its rows, so
// every workgroup ends and its peers get what they wait for; they stop waiting
// too once they see the fault, and the results are void.  (The row loop has no
// way out, so that it has no branch around loads.)  Launches that find the fault
// raised do nothing but tell the host, so that a solve ends.
#pragma once

#include "modap_device.hpp"
#include "sweep_split.hpp"
#include "sweep_wide.hpp"

namespace modap {

struct RelayArgs {
    SplitArgs s;             // A, b, nu, work, pd, r_out, part, scalars (one per band); ntiles
    int64_t tile;            // columns of a tile (the last may be shorter)
    uint64_t *words;         // [bands][kRelayRing][relay_row_words(ntiles)]
    uint32_t base;           // number of the band's row 0 in this launch
    uint32_t pad;
    int64_t timeout_ticks;
};

constexpr int kRelayThreads = 512;              // streaming threads
constexpr int kRelayRing = 16;
constexpr int kRelayRows = 4;                   // rows in registers: one in work, the others in flight
// Rows that a partial of y adds in one chain; the chains are added up beside
// it.  A band has as many rows as a CU streams in a sweep, twice those of the
// two phases: in one chain y of 16384 BF16 rows of 24000 was 14% further off than
// in two phases (rms, 1.19e-7 and 1.05e-7), in chains of 8 it is 21% closer
// (0.83e-7).  The 16 values more a thread are what the registers still hold.
constexpr int kRelayChain = 8;
constexpr int kRelayMaxTiles = 32;              // two exchanged words of four per lane
// Words of a row: of each tile the dots with x and v in two halves each, then
// the two halves of b.
__host__ __device__ constexpr int relay_row_words(int ntiles) { return ntiles * 4 + 2; }
constexpr int relay_chunks(int dt) { return dt == 2 ? 2 : 4; }   // 16-byte vectors per thread and row
constexpr int relay_depth(int dt) { return dt == 2 ? 8 : 4; }    // D
constexpr int relay_ahead(int dt) { return dt == 2 ? 3 : 1; }    // F
constexpr size_t relay_hold(int dt) {           // LDS that holds rows: 128 KiB
    return 16 * (size_t)kRelayThreads * (size_t)relay_chunks(dt) * (size_t)relay_depth(dt);
}
constexpr int64_t relay_tile(int dt) {          // columns of a tile at most
    return (int64_t)kRelayThreads * (dt == 0 ? 2 : dt == 1 ? 4 : 8) * relay_chunks(dt);
}

// A value that every lane holds, as the compiler can see: branches on it are
// scalar.
__device__ __forceinline__ double uniform(double v) { return lane_value(v, 0); }

template <int DT, bool HAS_V>
__global__ __launch_bounds__(kRelayThreads + 128) void sweep_relay(const RelayArgs ra) {
    using S = Store<DT>;
    using Acc = typename S::Acc;
    using T = typename S::T;
    constexpr int VEC = S::VEC, C = relay_chunks(DT), D = relay_depth(DT), F = relay_ahead(DT), P = kRelayRows;
    constexpr int NT = kRelayThreads, NW = NT / 64, CW = NT * VEC, AV = 16 / (int)sizeof(Acc);
    static_assert(kRelayChain % kRelayRows == 0 && (kRelayChain & (kRelayChain - 1)) == 0, "closed between passes");
    static_assert(D >= P && D >= F + 3 && kRelayRing >= 2 * D - 2, "ring and hold fit the pipeline");
    const SplitArgs &a = ra.s;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tile = (int)(blockIdx.x % (unsigned)a.ntiles), band = (int)(blockIdx.x / (unsigned)a.ntiles);
    const uint32_t fault = load_global(&a.pd.ctl->fault);   // (arrives with the state)
    const State st = sweep_state(a.pd, lane, blockIdx.x == 0 && tid == 0);
    if (a.check_status && st.status != ST_RUNNING) return;
    const bool apply_v = HAS_V && (st.vpend_valid || st.v_idx >= 0);
    const double s = a.pd.decide ? st.s : 0.0;   // step decided on the previous check

    const int64_t tile0 = (int64_t)tile * ra.tile;
    const int64_t width = min(ra.tile, a.ldA - tile0);
    const int64_t r0 = (int64_t)band * a.rows_per_band;
    const int64_t r1 = min(a.m, r0 + a.rows_per_band);
    const int R = (int)max((int64_t)0, r1 - r0);

    extern __shared__ __attribute__((aligned(16))) unsigned char hold_raw[];
    uint4 *hold = reinterpret_cast<uint4 *>(hold_raw);   // [D][C][NT]
    __shared__ Acc red[2][NW][2];
    __shared__ double wsh[2];
    __shared__ uint32_t gave_up;   // an earlier launch did; one reading for the whole workgroup
    if (tid < 2) wsh[tid] = 0.0;   // (what the first D iterations add)
    if (tid == 0) {
        gave_up = fault;
        if (fault && blockIdx.x == 0 && a.pd.progress) post_progress(a.pd.progress, a.pd.j - 1, ST_FAULT);
    }
    // row R-1 is added in iteration R-1+D; a multiple of F (the iterations past
    // the last row add nothing: their weights are zero)
    const int iters = (R + D + F - 1) / F * F;

    const int dots = a.ntiles * 4, nwords = relay_row_words(a.ntiles);
    uint64_t *mine = ra.words + (int64_t)band * kRelayRing * nwords;
    if (wave == NW + 1) {
        // ---- publishing wavefront: word q of this tile is the dot (q < 2) or
        // the translation's, low or high half; tile 0's words 4 and 5 are b
        const bool gives_b = HAS_V && tile == 0;
        double bnow = 0.0, bnext = 0.0;   // lane i: b of row 64 q + i, of this block of rows and the next
        if (gives_b && R > 0) bnext = a.b_in[r0 + min(lane, R - 1)];
        __syncthreads();
        if (gave_up) return;
        for (int t = 0; t < iters; ++t) {
            const int rp = t - 1;
            if (rp >= 0 && rp < R) {
                if (gives_b && (rp & 63) == 0) {
                    bnow = bnext;
                    if (rp + 64 < R) bnext = a.b_in[r0 + min(rp + 64 + lane, R - 1)];
                }
                const double bp = lane_value(bnow, rp & 63);
                if (lane < (gives_b ? 6 : 4)) {
                    double v = bp;
                    if (lane < 4) {
                        v = 0.0;
#pragma unroll
                        for (int w = 0; w < NW; ++w) v += (double)red[rp & 1][w][lane >> 1];
                    }
                    const uint64_t u = __builtin_bit_cast(uint64_t, v);
                    const uint32_t half = (lane & 1) ? (uint32_t)(u >> 32) : (uint32_t)u;
                    __hip_atomic_store(mine + (int64_t)(rp % kRelayRing) * nwords + (lane < 4 ? tile * 4 : dots - 4) + lane,
                                       ((uint64_t)(ra.base + (uint32_t)rp) << 32) | half, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            __syncthreads();
        }
        return;
    }
    if (wave == NW) {
        // ---- weighing wavefront
        const bool first_tile = tile == 0;
        int64_t h = 0;
        double dmax = 0.0, binf = 0.0, bkeep = 0.0, rkeep = 0.0, nkeep = 1.0;
        bool waits = true;
        // a lane's words of a row are lane and lane + 64 of the dots (clamped: a
        // lane past the last looks at that one too), and a half of b
        constexpr int NL = HAS_V ? 3 : 2;
        const int at[3] = {min(lane, dots - 1), min(lane + 64, dots - 1), dots + (lane & 1)};
        auto fetch = [&](int r, uint64_t (&w)[NL]) {
            uint64_t *row = mine + (int64_t)(r % kRelayRing) * nwords;
#pragma unroll
            for (int l = 0; l < NL; ++l) w[l] = __hip_atomic_load(row + at[l], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        };
        auto fresh = [&](const uint64_t (&w)[NL], int r) {
            bool all = true;
#pragma unroll
            for (int l = 0; l < NL; ++l) all &= (uint32_t)(w[l] >> 32) == ra.base + (uint32_t)r;
            return __all(all);
        };
        // Every iteration issues the same loads whether there is a row for them
        // or not, and a fetch only once the words in its
        // registers have been used: the compiler then counts which loads are
        // outstanding, and a fetch stays in flight over F iterations.  (A branch
        // around them, or a copy, became a wait for all of them.)
        uint64_t word[F][NL] = {};
        double bi[F] = {}, ni[F] = {};   // b (if not among the words) and ||a||^2 of the row, requested with them
        __syncthreads();
        if (gave_up) return;
        for (int t0 = 0; t0 < iters; t0 += F) {
#pragma unroll
            for (int k = 0; k < F; ++k) {
                const int t = t0 + k, rw = t - D + 1, rf = rw + F;
                const bool have = rw >= 0 && rw < R;
                double d = 0.0, td = 0.0, bb = HAS_V ? 0.0 : uniform(bi[k]);
                if (have) {
                    uint64_t w[NL];
#pragma unroll
                    for (int l = 0; l < NL; ++l) w[l] = word[k][l];
                    if (!fresh(w, rw) && waits) {
                        WaitClock wait;
                        do {
                            waits = __all(wait.goes_on(a.pd.ctl, ra.timeout_ticks));
                            fetch(rw, w);
                        } while (!fresh(w, rw) && waits);
                    }
                    // The row's dots over all tiles, in a fixed order: lanes 4q and
                    // 4q+2 put their two halves together, the quads are added inside
                    // each row of 16 lanes by rotations, then across the rows.  (One
                    // tile after another it is a chain of reads and adds that cost
                    // more than the rest of the iteration: n = 32000 took 3.6 ms.)
                    auto whole = [&](uint64_t v) -> double {   // (in even lanes)
                        const int own = (int)(uint32_t)v;
                        const int other = __builtin_amdgcn_update_dpp(0, own, 0xB1, 0xF, 0xF, true);   // lane ^ 1
                        return __hiloint2double(other, own);
                    };
                    auto dot_of = [&](uint64_t v, int first) { return first + (lane >> 2) < a.ntiles ? whole(v) : 0.0; };
                    double v = dot_of(w[0], 0);
                    if (dots > 64) v += dot_of(w[1], 16);
                    v += dpp_move<0x124>(v);   // the row rotated by 4 lanes
                    v += dpp_move<0x128>(v);   // and by 8
                    v = xor_add<32>(xor_add<16>(v));
                    d = lane_value(v, 0);
                    td = lane_value(v, 2);
                    if constexpr (HAS_V) bb = lane_value(whole(w[2]), 0);
                }
                const double nw = uniform(ni[k]);
                {
                    const int rc = max(0, min(rf, R - 1));
                    fetch(rc, word[k]);
                    if constexpr (!HAS_V) bi[k] = a.b_in[r0 + rc];
                    ni[k] = a.nu[r0 + rc];
                }
                double weight = 0.0;
                if (have) {
                    if (apply_v) bb += td;
                    const double r = d - bb;
                    weight = r > 0.0 ? r / nw : 0.0;
                    if (first_tile) {
                        // lane i keeps row 64 q + i; the counts are formed, and b
                        // and r written, for 64 rows at a time
                        if (lane == (rw & 63)) {
                            bkeep = bb;
                            rkeep = r;
                            nkeep = nw;
                        }
                        if ((rw & 63) == 63 || rw == R - 1) {
                            const int row = (rw & ~63) + lane;
                            if (row <= rw) {
                                binf = max_nan(binf, fabs(bkeep));
                                h += rkeep > 0.0 ? 1 : 0;
                                const double dist = rkeep / sqrt(nkeep);
                                dmax = rkeep > 0.0 ? max_nan(dmax, dist) : (rkeep != rkeep ? rkeep : dmax);
                                if (apply_v && a.b_out) a.b_out[r0 + row] = bkeep;
                                if (a.r_out) a.r_out[r0 + row] = rkeep;
                            }
                        }
                    }
                }
                if (lane == 0) wsh[rw & 1] = weight;
                __syncthreads();
            }
        }
        if (first_tile) {
            h = (int64_t)wave_total((double)h);   // an integer below 2^53: exact
            dmax = wave_max_nan(dmax);
            binf = wave_max_nan(binf);
            if (lane == 0) {
                a.h_part[band] = h;
                a.dmax_part[band] = dmax;
                a.binf_part[band] = binf;
            }
        }
        return;
    }

    // ---- streaming wavefronts
    const char *Ab = reinterpret_cast<const char *>(a.A) + tile0 * (int64_t)sizeof(T);
    const int64_t row_bytes = a.ldA * (int64_t)sizeof(T);
    const uint32_t range = (uint32_t)(width * (int64_t)sizeof(T));
    // Rows through a buffer resource each, whose range is the tile (columns
    // past it read as zeros); rows past the band re-read its last row, so
    // every iteration issues the same loads.
    auto load_row = [&](uint4 (&buf)[C], int r) {
        const __amdgpu_buffer_rsrc_t rr = row_resource(Ab + (r0 + max(0, min(r, R - 1))) * row_bytes, range);
#pragma unroll
        for (int c = 0; c < C; ++c) buf[c] = load_row_vec(rr, (uint32_t)((c * CW + tid * VEC) * (int)sizeof(T)));
    };
    uint4 buf[P][C];
    if (R > 0) {
#pragma unroll
        for (int k = 0; k < P; ++k) load_row(buf[k], k);
    }
    Acc xr[C][VEC], vr[C][VEC], yacc[C][VEC], ysum[C][VEC];
    const Acc *wx = reinterpret_cast<const Acc *>(a.work);
    const Acc *wv = wx + a.ldA;
    const Acc *wy = wx + 2 * a.ldA;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int64_t cc = (int64_t)c * CW + tid * VEC;
        const bool in = cc < width;
        const int64_t col = tile0 + (in ? cc : 0);
#pragma unroll
        for (int e = 0; e < VEC; e += AV) {
            const uint4 ux = *reinterpret_cast<const uint4 *>(wx + col + e);
            __builtin_memcpy(&xr[c][e], &ux, 16);
            if (HAS_V) {
                const uint4 uv = *reinterpret_cast<const uint4 *>(wv + col + e);
                __builtin_memcpy(&vr[c][e], &uv, 16);
            }
            if (s != 0.0) {
                Acc yv[AV];
                const uint4 uy = *reinterpret_cast<const uint4 *>(wy + col + e);
                __builtin_memcpy(yv, &uy, 16);
#pragma unroll
                for (int k = 0; k < AV; ++k) xr[c][e + k] = (Acc)step_point((double)xr[c][e + k], s, (double)yv[k]);
            }
        }
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            if (!in || !HAS_V) vr[c][e] = (Acc)0;
            if (!in) xr[c][e] = (Acc)0;
            yacc[c][e] = ysum[c][e] = (Acc)0;
        }
    }
    __syncthreads();
    if (gave_up) return;
    int place = 0;   // t % D, row t's place among the held rows
    auto add_held = [&](int t) {
        const double wd = uniform(wsh[(t - D) & 1]);
        if (wd == 0.0) return;
        const uint4 *slot = hold + (size_t)place * C * NT;
        const Acc w = (Acc)wd;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            Acc av[VEC];
            unpack<DT>(slot[c * NT + tid], av);
#pragma unroll
            for (int e = 0; e < VEC; ++e) yacc[c][e] = fma(w, av[e], yacc[c][e]);
        }
    };
    auto dot_and_hold = [&](const uint4 (&b)[C], int t) {
        uint4 *slot = hold + (size_t)place * C * NT;
        Acc d = (Acc)0, td = (Acc)0;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            Acc av[VEC];
            unpack<DT>(b[c], av);
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                d = fma(xr[c][e], av[e], d);
                if (HAS_V) td = fma(vr[c][e], av[e], td);
            }
            slot[c * NT + tid] = b[c];
        }
        d = wave_total(d);
        if (HAS_V) td = wave_total(td);
        if (lane == 0) {
            red[t & 1][wave][0] = d;
            red[t & 1][wave][1] = td;
        }
    };
    auto close_chain = [&]() {
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                ysum[c][e] += yacc[c][e];
                yacc[c][e] = (Acc)0;
            }
    };
    // (every pass of this loop issues the same loads, so that the compiler
    // counts exactly which of them a row still waits for)
    int t = 0;
    for (; t + P <= R; t += P) {
        if ((t & (kRelayChain - 1)) == 0) close_chain();
#pragma unroll
        for (int k = 0; k < P; ++k) {
            add_held(t + k);
            dot_and_hold(buf[k], t + k);
            load_row(buf[k], t + k + P);
            place = place + 1 < D ? place + 1 : 0;
            __syncthreads();
        }
    }
    // the last rows, already in registers, and the rows still held
#pragma unroll
    for (int k = 0; k < P; ++k) {
        if (t + k >= iters) break;
        add_held(t + k);
        if (t + k < R) dot_and_hold(buf[k], t + k);
        place = place + 1 < D ? place + 1 : 0;
        __syncthreads();
    }
    for (t += P; t < iters; ++t) {
        add_held(t);
        place = place + 1 < D ? place + 1 : 0;
        __syncthreads();
    }
    close_chain();
    Acc *part = reinterpret_cast<Acc *>(a.part) + (int64_t)band * a.ldPart + tile0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int64_t cc = (int64_t)c * CW + tid * VEC;
        if (cc >= width) continue;
#pragma unroll
        for (int e = 0; e < VEC; e += AV) {
            uint4 w;
            __builtin_memcpy(&w, &ysum[c][e], 16);
            *reinterpret_cast<uint4 *>(part + cc + e) = w;
        }
    }
}

}  // namespace modap
