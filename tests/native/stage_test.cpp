// Test driver of the server's staging memory (paper_2003_09956_amd/csrc/stage_pool.hpp)
// over streams that come and go.  No device is needed: the runtime's calls are
// defined here, and an event that is asked after its stream has gone is a
// failed check.  Exits non-zero on the first failed check.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <set>

#include "stage_pool.hpp"

static int failures = 0, refuse = 0, held = 0;
#define EXPECT(cond)                                                                          \
    do {                                                                                      \
        if (!(cond)) {                                                                        \
            std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #cond);     \
            ++failures;                                                                       \
        }                                                                                     \
    } while (0)

struct Ev {
    hipStream_t on;
    bool done;
};
static std::map<hipEvent_t, Ev> events;
static std::set<hipStream_t> streams;
static size_t names = 0;

static hipStream_t open_stream() { return *streams.insert(reinterpret_cast<hipStream_t>(++names * 16)).first; }

extern "C" {
hipError_t hipMalloc(void **p, size_t bytes) {
    if (refuse) return hipErrorOutOfMemory;
    *p = std::malloc(bytes);
    ++held;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    std::free(p);
    --held;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    if (refuse) return hipErrorOutOfMemory;
    *e = reinterpret_cast<hipEvent_t>(++names * 16);
    events[*e] = Ev{nullptr, true};
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
    EXPECT(events.erase(e) == 1);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    EXPECT(events.count(e) && streams.count(s));
    events[e] = Ev{s, false};
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
    EXPECT(events.count(e) && streams.count(events[e].on));
    return events[e].done ? hipSuccess : hipErrorNotReady;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
    EXPECT(events.count(e) && streams.count(events[e].on));
    events[e].done = true;
    return hipSuccess;
}
}

static modap_host::Stage *take(modap_host::StagePool &p, size_t bytes) {
    modap_host::Stage *t = nullptr;
    const char *what = "";
    EXPECT(p.take(bytes, &t, &what) == hipSuccess && t && t->p && t->used && !t->busy && t->size >= bytes);
    return t;
}

int main() {
    modap_host::StagePool pool;
    const hipStream_t a = open_stream(), b = open_stream();
    modap_host::Stage *t = take(pool, 100);
    void *const first = t->p;
    EXPECT(pool.used(t, a) == hipSuccess);
    t = take(pool, 100);   // the first is not free: its update has not run
    EXPECT(t->p != first && held == 2);
    EXPECT(pool.used(t, b) == hipSuccess);
    for (auto &e : events)
        if (e.second.on == a) e.second.done = true;
    t = take(pool, 100);   // now it is
    EXPECT(t->p == first && held == 2);
    EXPECT(pool.used(t, a) == hipSuccess);
    // a's work has run and it goes: the stage on it is free, and no event of it is left to ask
    pool.end_stream(a);
    streams.erase(a);
    t = take(pool, 100);
    EXPECT(t->p == first && held == 2 && events.size() == 2);
    EXPECT(pool.used(t, b) == hipSuccess);
    take(pool, 1 << 21);   // larger than either
    EXPECT(held == 3);
    // refused memory and a refused event: nothing half made
    pool.end_stream(b);
    streams.erase(b);
    EXPECT(events.size() == 1);
    refuse = 1;
    const char *what = "";
    EXPECT(pool.take(1 << 22, &t, &what) == hipErrorOutOfMemory && !t && held == 3);
    EXPECT(pool.take(100, &t, &what) == hipErrorOutOfMemory && !t && held == 3);
    refuse = 0;
    const hipStream_t c = open_stream();
    EXPECT(pool.used(take(pool, 100), c) == hipSuccess);
    pool.destroy();
    EXPECT(held == 0 && events.empty());
    if (failures) return 1;
    std::puts("all staging checks passed");
    return 0;
}
