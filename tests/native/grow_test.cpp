// Test driver of the library's growing device buffers
// (paper_2003_09956_amd/csrc/host_common.hpp) over an allocator that can refuse.  No device is
// needed: the runtime's calls are defined here.  Exits non-zero on the first
// failed check.
#include <cstdio>
#include <cstdlib>

#include "host_common.hpp"

static int failures = 0, refuse = 0, held = 0;
#define EXPECT(cond)                                                                          \
    do {                                                                                      \
        if (!(cond)) {                                                                        \
            std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #cond);     \
            ++failures;                                                                       \
        }                                                                                     \
    } while (0)

extern "C" {
hipError_t hipMalloc(void **p, size_t bytes) {
    if (refuse) return hipErrorOutOfMemory;   // *p is left as it is
    *p = std::malloc(bytes);
    ++held;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    std::free(p);
    --held;
    return hipSuccess;
}
}

int main() {
    using modap_host::grow_dev;
    double *p = nullptr;
    void *v = nullptr;
    size_t cap = 0, bytes = 0;
    EXPECT(grow_dev(p, cap, 0, sizeof *p) == hipSuccess && !p && cap == 0);
    EXPECT(grow_dev(p, cap, 100, sizeof *p) == hipSuccess && p && cap == 100);
    p[99] = 1.0;
    double *const first = p;
    EXPECT(grow_dev(p, cap, 50, sizeof *p) == hipSuccess && p == first && cap == 100);
    refuse = 1;
    EXPECT(grow_dev(p, cap, 100, sizeof *p) == hipSuccess && p == first);   // nothing to ask for
    EXPECT(grow_dev(p, cap, 101, sizeof *p) == hipErrorOutOfMemory);
    // no buffer is no capacity: a call that needs less than was held before must ask again
    EXPECT(!p && cap == 0 && held == 0);
    EXPECT(grow_dev(p, cap, 50, sizeof *p) == hipErrorOutOfMemory && !p && cap == 0);
    EXPECT(grow_dev(v, bytes, 7, 1) == hipErrorOutOfMemory && !v && bytes == 0);
    refuse = 0;
    EXPECT(grow_dev(p, cap, 50, sizeof *p) == hipSuccess && p && cap == 50);
    EXPECT(grow_dev(v, bytes, 7, 1) == hipSuccess && v && bytes == 7 && held == 2);
    p[49] = 2.0;
    modap_host::free_dev(p);
    modap_host::free_dev(v);
    EXPECT(held == 0 && !p && !v);
    if (failures) return 1;
    std::puts("all buffer checks passed");
    return 0;
}
