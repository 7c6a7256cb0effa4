// What the host reads back at the end of a call, written by the device into
// host memory (pinned, mapped and coherent) in place of copies.
//
// A copy to pageable host memory costs the host about 19 us, one to pinned
// memory 11 us, and waiting for the stream 11 us even behind an empty kernel;
// a kernel that writes the result itself and then a sequence number is seen
// by a polling host 5-6 us after its launch.  A batch_query of 256 doubles
// and a state took 35 us with three pageable copies.
#pragma once

#include <hip/hip_runtime.h>
#include <immintrin.h>

#include <atomic>
#include <cstring>
#include <stdint.h>

#include "modap_device.hpp"

namespace modap {

// The part with a fixed layout (one per context, batch).
struct alignas(128) HostView {
    State st;               // a committed state
    Totals tot;             // the totals of a stateless sweep
    uint64_t progress;      // solve: (settled check + 1) << 8 | its status, written by the next sweep
    uint32_t fault;         // a resident launch gave up waiting
    uint32_t pad32;
    uint64_t pad0;
    alignas(128) uint32_t seq;   // the last result that is complete
};

// What the checks of a system's data report: the first bad row (see
// row_norms) and whether b or x has a non-finite entry.  Adjacent, so that one
// request reads both back.
struct DataChecks {
    unsigned long long bad;
    unsigned long long flag;
};

struct PublishArgs {
    const State *st;        // or null
    const uint32_t *fault;  // or null
    const Totals *tot;      // or null
    const double *src[2];
    double *dst[2];         // host staging or caller memory, count[k] doubles each
    int64_t count[2];
    HostView *view;
    uint32_t *arrived;      // zero between launches
    uint32_t seq;
    uint32_t pad;
};

// Called by every thread of a workgroup after its writes: the last workgroup
// of the grid announces result `seq`.  Each thread's writes are ordered before
// its workgroup's arrival, and the arrivals before the announcement.
__device__ __forceinline__ void announce(HostView *view, uint32_t *arrived, uint32_t seq, uint32_t workgroups) {
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x != 0) return;
    if (workgroups > 1) {
        if (__hip_atomic_fetch_add(arrived, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) != workgroups - 1) return;
        __hip_atomic_store(arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __hip_atomic_store(&view->seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Vectors and one state to the host (latency bound: one workgroup up to
// kPublishAlone doubles, else 32).
constexpr int64_t kPublishAlone = 4096;
static __global__ __launch_bounds__(256) void publish(const PublishArgs a) {
    const int64_t first = (int64_t)blockIdx.x * 256 + threadIdx.x, step = (int64_t)gridDim.x * 256;
#pragma unroll
    for (int k = 0; k < 2; ++k)
        for (int64_t i = first; i < a.count[k]; i += step) a.dst[k][i] = a.src[k][i];
    if (blockIdx.x == 0 && threadIdx.x < sizeof(State) / 8) {
        if (a.st)
            reinterpret_cast<uint64_t *>(&a.view->st)[threadIdx.x] = reinterpret_cast<const uint64_t *>(a.st)[threadIdx.x];
        if (a.tot && threadIdx.x < sizeof(Totals) / 8)
            reinterpret_cast<uint64_t *>(&a.view->tot)[threadIdx.x] =
                reinterpret_cast<const uint64_t *>(a.tot)[threadIdx.x];
        if (a.fault && threadIdx.x == 0) a.view->fault = *a.fault;
    }
    announce(a.view, a.arrived, a.seq, gridDim.x);
}

}  // namespace modap

namespace modap_host {

// The host side: the view, its device address, and staging for vectors.
struct Readback {
    modap::HostView *view = nullptr;       // host address
    modap::HostView *dev = nullptr;        // device address of the same memory
    uint32_t *arrived = nullptr;           // device counter
    uint32_t seq = 0;
    double *buf = nullptr, *buf_dev = nullptr;
    size_t cap = 0;                        // doubles

    hipError_t create(hipStream_t s) {
        hipError_t e = hipHostMalloc(&view, sizeof(modap::HostView), hipHostMallocMapped);
        if (e == hipSuccess) e = hipHostGetDevicePointer(reinterpret_cast<void **>(&dev), view, 0);
        if (e == hipSuccess) e = hipMalloc(&arrived, sizeof(uint32_t));
        if (e == hipSuccess) e = hipMemsetAsync(arrived, 0, sizeof(uint32_t), s);
        if (e == hipSuccess) *view = modap::HostView{};
        return e;
    }
    void destroy() {
        if (view) (void)hipHostFree(view);
        if (buf) (void)hipHostFree(buf);
        if (arrived) (void)hipFree(arrived);
        view = dev = nullptr;
        buf = buf_dev = nullptr;
        arrived = nullptr;
        cap = 0;
    }
    // Staging up to this many doubles (8 MiB): above, a copy costs little
    // next to the transfer itself.
    static constexpr int64_t kMaxStaged = int64_t(1) << 20;
    hipError_t reserve(int64_t doubles) {
        if ((size_t)doubles <= cap) return hipSuccess;
        size_t want = 4096;
        while (want < (size_t)doubles) want *= 2;
        if (buf) (void)hipHostFree(buf);   // (no result is outstanding: every call that stages one waits for it)
        buf = buf_dev = nullptr;
        cap = 0;
        hipError_t e = hipHostMalloc(&buf, want * sizeof(double), hipHostMallocMapped);
        if (e == hipSuccess) e = hipHostGetDevicePointer(reinterpret_cast<void **>(&buf_dev), buf, 0);
        if (e == hipSuccess) cap = want;
        return e;
    }
    // Wait for the result just queued on `s` (number `seq`).  The host polls
    // for a few milliseconds, then leaves the waiting to the runtime, which
    // also reports a failed launch.  Every 256th result the stream is
    // synchronised, so that the runtime retires what it holds for it.
    hipError_t wait(hipStream_t s) {
        volatile uint32_t *p = &view->seq;
        for (uint32_t spin = 0; *p != seq; ++spin) {
            if (spin == kSpins) {
                const hipError_t e = hipStreamSynchronize(s);
                return e == hipSuccess && *p != seq ? hipErrorUnknown : e;
            }
            _mm_pause();
        }
        std::atomic_thread_fence(std::memory_order_acquire);
        return (seq & 0xff) == 0 ? hipStreamSynchronize(s) : hipSuccess;
    }
    static constexpr uint32_t kSpins = 1u << 17;
    // Queue `publish` for what `a` names and wait for it.
    hipError_t run(modap::PublishArgs a, hipStream_t s) {
        a.view = dev;
        a.arrived = arrived;
        a.seq = ++seq;
        const int grid = a.count[0] + a.count[1] <= modap::kPublishAlone ? 1 : 32;
        hipLaunchKernelGGL(modap::publish, dim3(grid), dim3(256), 0, s, a);
        const hipError_t e = hipGetLastError();
        return e == hipSuccess ? wait(s) : e;
    }
};

// The checks of a system's data, once the work queued on `s` is done.
inline hipError_t read_checks(Readback &rb, const modap::DataChecks *checks, hipStream_t s, modap::DataChecks *out) {
    static_assert(sizeof(modap::DataChecks) == 2 * sizeof(double), "read back as two doubles");
    hipError_t e = rb.reserve(2);
    if (e != hipSuccess) return e;
    modap::PublishArgs a{};
    a.src[0] = reinterpret_cast<const double *>(checks);
    a.dst[0] = rb.buf_dev;
    a.count[0] = 2;
    e = rb.run(a, s);
    if (e == hipSuccess) std::memcpy(out, rb.buf, sizeof *out);
    return e;
}

}  // namespace modap_host
