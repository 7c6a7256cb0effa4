// Test driver of the rule that paces a solve
// (paper_2003_09956_amd/csrc/host_common.hpp).  No device is needed.  Exits
// non-zero on the first failed check.
#include <cstdio>

#include "host_common.hpp"

static int failures = 0;
#define EXPECT(cond)                                                                          \
    do {                                                                                      \
        if (!(cond)) {                                                                        \
            std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #cond);     \
            ++failures;                                                                       \
        }                                                                                     \
    } while (0)

// A solve whose host queues an iteration in `launch` time units (the device
// takes 1 each) but is held up for `hitch` units every `every` iterations.
// Returns the units that the device spent waiting in the second half.
static double waited(double launch, double hitch, int every, int steps, int64_t *most) {
    double host = 0.0, device = 0.0, idle = 0.0;
    int64_t ahead = 4, queued = 0, settled = 0;
    double ends[1 << 14];   // when each iteration ends on the device
    *most = ahead;
    while (queued < steps) {
        for (; settled < queued - 1 && ends[settled] <= host; ++settled) {
        }
        ahead = modap_host::solve_ahead_after(ahead, queued - settled, settled);
        if (ahead > *most) *most = ahead;
        if (queued - settled >= ahead) {
            host = host > ends[settled] ? host : ends[settled];
            continue;
        }
        host += launch + (queued % every == every - 1 ? hitch : 0.0);
        if (host > device) {
            if (queued > steps / 2) idle += host - device;
            device = host;
        }
        device += 1.0;
        ends[queued++] = device;
    }
    return idle;
}

int main() {
    using modap_host::kMostAhead;
    using modap_host::solve_ahead_after;
    int64_t most = 0;
    for (int64_t a = 1; a <= kMostAhead; a *= 2)
        for (int64_t left = 0; left <= a; ++left)
            for (int64_t settled : {0, 1, 31, 32, 100, 512, 100000}) {
                const int64_t b = solve_ahead_after(a, left, settled);
                EXPECT(b == a || b == 2 * a);
                EXPECT(b <= kMostAhead && (b == a || b <= settled / 4));
                if (4 * left > a) EXPECT(b == a);
            }
    EXPECT(solve_ahead_after(2, 1, 1000) == 2);   // two long iterations: one left is what it should be
    // a host that keeps up never queues more; nor does one in a short solve
    EXPECT(waited(0.5, 0.0, 100, 8000, &most) == 0.0 && most == 4);
    (void)waited(0.5, 30.0, 8, 31, &most);
    EXPECT(most == 4);
    // one that is held up now and then for longer than four iterations gets in front again
    EXPECT(waited(0.5, 15.0, 100, 8000, &most) == 0.0 && most > 4);
    EXPECT(waited(0.5, 30.0, 200, 8000, &most) == 0.0 && most <= kMostAhead);
    if (failures) return 1;
    std::puts("all pacing checks passed");
    return 0;
}
