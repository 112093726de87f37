// Driver for the pinned result slots (built by tests/test_host_result.py for the
// CPU): capi.cpp over a HIP runtime of its own, whose stream waits fail on demand.
#include "capi.cpp"

#include <cstdio>
#include <cstdlib>
#include <set>
#include <vector>

static hipError_t g_wait = hipSuccess;
static int g_copies = 0;

extern "C" {
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned) { *p = calloc(1, bytes); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void **d, void *p, unsigned) { *d = p; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return g_wait; }
hipError_t hipMemcpyAsync(void *, const void *, size_t, hipMemcpyKind, hipStream_t) { ++g_copies; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return ""; }
}

#define CHECK(c) do { if (!(c)) { printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)

using namespace mcmie;

// One call: a slot, a kernel that would write `v` to it, the wait.
static double *call(double v, double *out, bool launch = true)
{
    HostResult host;
    if (!host) return nullptr;
    if (!launch) return (double *)out;   // (an early return before anything was handed out)
    double *at = host.data();
    at[0] = v;
    (void)wait_result(out, 1, nullptr, host, nullptr);
    return at;
}

int main()
{
    double out[1] = {0.0};
    // Sound waits: one slot serves any number of calls, and so do early returns.
    double *first = call(1.0, out);
    CHECK(first && out[0] == 1.0);
    for (int i = 0; i < 200; ++i) CHECK(call(2.0 + i, out) == first && out[0] == 2.0 + i);
    for (int i = 0; i < 200; ++i) CHECK(call(0.0, out, false));
    CHECK(call(5.0, out) == first);
    // A failed wait: its slot is no later call's, while the kernel may still write.
    g_wait = hipErrorUnknown;
    double *lost = call(7.0, out);
    CHECK(lost == first && out[0] == 5.0);
    g_wait = hipSuccess;
    for (int i = 0; i < 200; ++i) {
        double *at = call(8.0, out);
        CHECK(at && at != lost && out[0] == 8.0);
        lost[0] = -1.0;   // the late write
        CHECK(out[0] == 8.0);
    }
    // All slots lost: calls copy.
    g_wait = hipErrorUnknown;
    std::set<double *> taken{lost};
    for (int i = 0; i < 63; ++i) CHECK(taken.insert(call(9.0, out)).second);
    g_wait = hipSuccess;
    HostResult none;
    CHECK(!none && wait_result(out, 1, out, none, nullptr) == hipSuccess && g_copies == 1);
    printf("OK\n");
    return 0;
}
