// Error reporting and version entry points of the C ABI.
#include "common.hpp"

#include <atomic>
#include <cstring>
#include <mutex>

namespace mcmie {

static thread_local char g_msg[512] = "";

int fail(int code, const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_msg, sizeof g_msg, fmt, ap);
    va_end(ap);
    return code;
}

void clear_error() { g_msg[0] = '\0'; }

int device_cu_count(int *out)
{
    static std::mutex mu;
    static int cached[64] = {0};
    int dev = 0;
    MC_HIP_CHECK(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) return fail(MC_EDEVICE, "device index %d out of range", dev);
    std::lock_guard<std::mutex> lock(mu);
    if (cached[dev] == 0) {
        int n = 0;
        MC_HIP_CHECK(hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev));
        cached[dev] = n > 0 ? n : 1;
    }
    *out = cached[dev];
    return MC_OK;
}

static std::atomic<uint64_t> g_free{~0ull};   // free slots of g_pinned
static double *g_pinned = nullptr;            // 64 x kHostResult doubles
static std::once_flag g_pinned_once;

HostResult::HostResult() : slot_(-1)
{
    std::call_once(g_pinned_once, [] {
        void *p = nullptr, *dev = nullptr;
        const size_t bytes = 64 * kHostResult * sizeof(double);
        if (hipHostMalloc(&p, bytes, hipHostMallocPortable | hipHostMallocMapped) != hipSuccess ||
            hipHostGetDevicePointer(&dev, p, 0) != hipSuccess || dev != p) {
            (void)hipGetLastError();
            return;
        }
        g_pinned = (double *)p;
    });
    if (!g_pinned) return;
    uint64_t free = g_free.load(std::memory_order_relaxed);
    while (free != 0) {
        const int i = __builtin_ctzll(free);
        if (g_free.compare_exchange_weak(free, free & ~(1ull << i), std::memory_order_acquire)) {
            slot_ = i;
            return;
        }
    }
}

HostResult::~HostResult()
{
    if (slot_ >= 0 && !lent_) g_free.fetch_or(1ull << slot_, std::memory_order_release);
}

double *HostResult::data()
{
    lent_ = true;
    return g_pinned + slot_ * kHostResult;
}

hipError_t wait_result(double *out, int n, const double *result, HostResult &host, hipStream_t st)
{
    if (!host) {
        const hipError_t e = hipMemcpyAsync(out, result, n * sizeof(double), hipMemcpyDeviceToHost, st);
        if (e != hipSuccess) return e;
    }
    const hipError_t e = hipStreamSynchronize(st);
    if (e == hipSuccess && host) {
        std::memcpy(out, host.data(), n * sizeof(double));
        host.settle();
    }
    return e;
}

}  // namespace mcmie

extern "C" const char *mc_last_error(void) { return mcmie::g_msg; }

extern "C" int mc_version(void) { return 400; }   // 0.4.0
