// Host-side helpers shared by the single-system and the batched halves of the
// library: device selection, error reporting into a context's message, and
// storage-type sizes.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <initializer_list>
#include <string>

#include "modap.h"
#include "validate.hpp"

namespace modap_host {

// Make `d` the current device for the guard's lifetime.
struct DeviceGuard {
    int prev = -1;
    explicit DeviceGuard(int d) {
        if (hipGetDevice(&prev) != hipSuccess) prev = -1;
        if (prev != d) (void)hipSetDevice(d);
    }
    ~DeviceGuard() {
        int cur = -1;
        if (prev >= 0 && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
    }
};

// Record `msg` as the context's last error and return `st` (any context type
// with a std::string member `err`).
template <typename Ctx>
modap_status fail(Ctx *c, modap_status st, const std::string &msg) {
    if (c) c->err = msg;
    return st;
}

// (The runtime keeps the error for whoever asks next, and the next launch of
// this thread, ours or another library's, would report it for its own.)
template <typename Ctx>
modap_status hip_fail(Ctx *c, hipError_t e, const char *what) {
    (void)hipGetLastError();
    if (e == hipErrorOutOfMemory) return fail(c, MODAP_E_NOMEM, std::string(what) + ": out of device memory");
    return fail(c, MODAP_E_DEVICE, std::string(what) + ": " + hipGetErrorString(e));
}

// Whether an asynchronous copy from host memory `p` reads it only when the
// stream comes to it: from pinned memory it does, from pageable memory the
// runtime has read it when the call returns.
inline bool read_later(const void *p) {
    hipPointerAttribute_t at{};
    if (!p || hipPointerGetAttributes(&at, p) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return at.type == hipMemoryTypeHost || at.type == hipMemoryTypeManaged;
}

// The caller's host inputs of a call are the caller's again when it returns: wait
// for the copies out of them, if there are any that the stream has still to come
// to.  (Nothing can be waited for under capture; a replay reads them again.)
inline hipError_t inputs_read(hipStream_t s, std::initializer_list<const void *> inputs) {
    for (const void *p : inputs)
        if (read_later(p)) {
            hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
            if (hipStreamIsCapturing(s, &cap) != hipSuccess) (void)hipGetLastError();
            return cap == hipStreamCaptureStatusNone ? hipStreamSynchronize(s) : hipSuccess;
        }
    return hipSuccess;
}

inline size_t elem_size(int dt) { return dt == 0 ? 8 : dt == 1 ? 4 : 2; }
inline size_t acc_size(int dt) { return dt == 0 ? 8 : 4; }
inline int vec_elems(int dt) { return 16 / (int)elem_size(dt); }

template <typename P>
void free_dev(P *&p) {
    if (p) (void)hipFree((void *)p);
    p = nullptr;
}

// A device buffer of at least `count` elements of `each` bytes, its contents
// not kept.  A failure leaves no buffer and a capacity of none, so that the next
// call, which may need less, asks again.
template <typename P>
hipError_t grow_dev(P *&p, size_t &cap, size_t count, size_t each) {
    if (count <= cap) return hipSuccess;
    free_dev(p);
    cap = 0;
    const hipError_t e = hipMalloc(reinterpret_cast<void **>(&p), count * each);
    if (e == hipSuccess)
        cap = count;
    else
        p = nullptr;
    return e;
}

// How many iterations a solve keeps queued when it sees that `left` of the
// `ahead` are still to run, `settled` being behind it: twice as many if no more
// than a quarter are left, up to kMostAhead and to a quarter of those behind (a
// stop leaves that many queued in vain).  A host that has fallen behind (a launch
// that takes long, a core that is shared) never gets in front again with few
// queued: with 4 throughout, in every other process solves of FP32 1000 x 4000
// took 11.4 us an iteration for 10.6, of 520 x 2000 10.4 for 9.4; up to 16 were
// not enough.
constexpr int64_t kMostAhead = 64;
inline int64_t solve_ahead_after(int64_t ahead, int64_t left, int64_t settled) {
    return 4 * left <= ahead && 8 * ahead <= settled && ahead < kMostAhead ? 2 * ahead : ahead;
}

// Several arrays in one device allocation (of each system, the vectors and
// small results): an allocation and a release each time a system comes and
// goes, in place of a dozen.
struct Pieces {
    static constexpr int kMax = 20;
    void **at[kMax];
    size_t off[kMax], total = 0;
    int count = 0;
    template <typename P>
    void add(P *&p, size_t bytes) {
        at[count] = reinterpret_cast<void **>(&p);
        off[count++] = total;
        total += (bytes + 255) / 256 * 256;
    }
    hipError_t alloc(void *&base) {
        const hipError_t e = hipMalloc(&base, total);
        if (e != hipSuccess) base = nullptr;
        for (int k = 0; e == hipSuccess && k < count; ++k) *at[k] = static_cast<char *>(base) + off[k];
        return e;
    }
};

}  // namespace modap_host

#define HIP_TRY(c, expr)                                                \
    do {                                                                \
        hipError_t e_ = (expr);                                         \
        if (e_ != hipSuccess) return ::modap_host::hip_fail((c), e_, #expr); \
    } while (0)

#define LAUNCH_TRY(c, what)                                             \
    do {                                                                \
        hipError_t e_ = hipGetLastError();                              \
        if (e_ != hipSuccess) return ::modap_host::hip_fail((c), e_, what); \
    } while (0)
