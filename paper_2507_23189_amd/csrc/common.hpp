// Host-side plumbing shared by the library's entry points: the thread-local
// error message behind mc_last_error(), HIP status checks, device queries.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdio>

#include "mcmie.h"

namespace mcmie {

// Records a formatted message for mc_last_error() and returns `code`.
int fail(int code, const char *fmt, ...);

// Clears the calling thread's message (start of every entry point).
void clear_error();

#define MC_HIP_CHECK(expr)                                                          \
    do {                                                                            \
        hipError_t e_ = (expr);                                                     \
        if (e_ != hipSuccess)                                                       \
            return ::mcmie::fail(MC_EDEVICE, "%s failed: %s", #expr,                \
                                 hipGetErrorString(e_));                            \
    } while (0)

// A kernel's scalar results on their way to the host: kHostResult doubles of
// pinned memory that every GPU writes to directly, so that a call that waits for
// its results needs no copy (a copy kernel and its gap, 8 to 10 of the 48 us of a
// small table build).  The library holds 64 of them until the process ends, each
// used by one call at a time; false when none is free or the memory cannot be
// had, and the call copies.  A slot whose address a call has handed to a kernel is
// free again only when wait_result has waited for the stream: where that fails (while
// another stream captures in global mode, say) the kernel may still be about to write
// to it, and the slot stays taken.
constexpr int kHostResult = 16;
class HostResult {
public:
    HostResult();
    ~HostResult();
    HostResult(const HostResult &) = delete;
    HostResult &operator=(const HostResult &) = delete;
    explicit operator bool() const { return slot_ >= 0; }
    double *data();   // for a kernel to write to
    // The stream has been waited for: no kernel writes to the slot any more.
    void settle() { lent_ = false; }

private:
    int slot_;
    bool lent_ = false;
};
// Wait for the stream and fetch n results written to `result` (host's, or
// device memory).
hipError_t wait_result(double *out, int n, const double *result, HostResult &host, hipStream_t st);

// Compute units of the current device (cached per device).
int device_cu_count(int *out);

}  // namespace mcmie
