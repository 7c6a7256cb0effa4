// Device memory for the inputs of updates, reusable once the update that read
// it has run (the server's; see modap_server_update).
#pragma once

#include <hip/hip_runtime.h>

#include <vector>

namespace modap_host {

struct Stage {
    void *p = nullptr;
    size_t size = 0;
    hipEvent_t used = nullptr;   // null: none recorded since the last end of its stream
    hipStream_t on = nullptr;    // where `used` was recorded last
    bool busy = false;
};

struct StagePool {
    std::vector<Stage> stages;

    // A stage of at least `bytes` whose last update has run (the pool grows when
    // none is free), valid until the next call; *what says which call failed.
    hipError_t take(size_t bytes, Stage **out, const char **what) {
        *out = nullptr;
        for (Stage &t : stages) {
            if (t.busy) {
                const hipError_t e = hipEventQuery(t.used);
                if (e == hipSuccess) {
                    t.busy = false;
                } else {
                    (void)hipGetLastError();   // (also "not ready", which is no error)
                    if (e != hipErrorNotReady) return *what = "hipEventQuery", e;
                }
            }
            if (!t.busy && t.size >= bytes) return event(t, out, what);
        }
        Stage t;
        t.size = (bytes + (1u << 20) - 1) / (1u << 20) * (1u << 20);
        if (const hipError_t e = hipMalloc(&t.p, t.size)) {
            (void)hipGetLastError();
            return *what = "hipMalloc", e;
        }
        stages.push_back(t);
        return event(stages.back(), out, what);
    }

    // What was queued on `stream` up to now reads the stage.
    hipError_t used(Stage *t, hipStream_t stream) {
        const hipError_t e = hipEventRecord(t->used, stream);
        t->on = stream;
        t->busy = true;
        return e;
    }

    // `stream`, whose work has run, is about to be destroyed.  An event must not
    // outlive the stream it was recorded on: the runtime looks at that stream
    // when the event is asked or waited for, and a server closed after it had
    // served many long requests at once left "operation not permitted when
    // stream is capturing" for the next caller of the runtime to find.
    void end_stream(hipStream_t stream) {
        for (Stage &t : stages)
            if (t.used && t.on == stream) {
                drop_event(t);
                t.busy = false;
            }
    }

    void destroy() {
        for (Stage &t : stages) {
            if (t.used) drop_event(t);
            (void)hipFree(t.p);
        }
        stages.clear();
    }

private:
    hipError_t event(Stage &t, Stage **out, const char **what) {
        if (!t.used) {
            const hipError_t e = hipEventCreateWithFlags(&t.used, hipEventDisableTiming);
            if (e != hipSuccess) {
                (void)hipGetLastError();
                t.used = nullptr;
                return *what = "hipEventCreateWithFlags", e;
            }
            t.on = nullptr;
        }
        *out = &t;
        return hipSuccess;
    }
    static void drop_event(Stage &t) {
        if (t.on) (void)hipEventSynchronize(t.used);
        (void)hipEventDestroy(t.used);
        t.used = nullptr;
        t.on = nullptr;
    }
};

}  // namespace modap_host
