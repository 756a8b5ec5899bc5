// Host-side pieces shared by the library's source files: the calling
// thread's error text, HIP error checks, the per-launch event profiler,
// launch-size helpers and the exception guard of the exported calls.
#pragma once

#include <hip/hip_runtime.h>
#include <rocprofiler-sdk-roctx/roctx.h>

#include <cstddef>
#include <cstdint>
#include <exception>

#include "mpt.h"

namespace mptlib {

// Sets the calling thread's error text (printf format); returns status.
int fail(int status, const char *fmt, ...);
void clear_error();
const char *error_text();

// While profiling is on (mpt_profile_begin), records HIP events on the
// caller's stream around one launch, under `name`, with `work` algorithmic
// units.
class LaunchScope {
  public:
    LaunchScope(const char *name, double work, hipStream_t s);
    ~LaunchScope();
    LaunchScope(const LaunchScope &) = delete;
    LaunchScope &operator=(const LaunchScope &) = delete;

  private:
    hipStream_t s_;
    bool active_ = false;
    hipEvent_t a_{}, b_{};
    const char *name_;
    double work_;
};

// A named roctx range around one phase of an exported call (visible to
// rocprofv3 --marker-trace; a no-op without a profiler).
class Range {
  public:
    explicit Range(const char *name) { roctxRangePushA(name); }
    ~Range() { roctxRangePop(); }
    Range(const Range &) = delete;
    Range &operator=(const Range &) = delete;
};

// A block of pinned host memory that kernels read and write directly. From a
// fixed pool (32 blocks, one allocation, made at the first use and kept: a
// block goes back when its HostSlot ends); a mutex guards the pool, so that
// calls on any threads, streams and devices may hold one each. ptr() is null
// when all are taken, when the allocation failed and while s is being captured
// (a recorded kernel must not keep the block's address): callers then copy.
class HostSlot {
  public:
    static constexpr size_t kBytes = 16384;
    explicit HostSlot(hipStream_t s);
    ~HostSlot();
    char *ptr() const { return ptr_; }
    // after an error, launches that use the block may be queued on s: it goes
    // back when they are over, or never if that cannot be waited for
    void settle(hipStream_t s) {
        if (ptr_ && hipStreamSynchronize(s) != hipSuccess) ptr_ = nullptr;
    }
    HostSlot(const HostSlot &) = delete;
    HostSlot &operator=(const HostSlot &) = delete;

  private:
    char *ptr_ = nullptr;
};

// Copies bytes (a multiple of 4) of device memory to ordinary host memory
// after the work queued on s, and waits for it. Up to HostSlot::kBytes go
// through a pinned block that a kernel writes: launch and wait take 15 us on
// an idle stream where hipMemcpyAsync to pageable memory and the wait take 22
// (11 is the launch and the wait alone).
// pinned = false: a plain copy and wait, for calls that must not allocate.
hipError_t read_back(void *dst, const void *src, size_t bytes, hipStream_t s, bool pinned = true);

inline int grid_for(int64_t n, int threads, int cap = 8192) {
    int64_t g = (n + threads - 1) / threads;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

inline size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

// Runs the body of an exported call: a C++ exception never crosses the C ABI,
// it becomes MPT_E_INTERNAL with its text.
template <class F>
inline int guarded(const char *where, F &&body) noexcept {
    try {
        return body();
    } catch (const std::exception &e) {
        return fail(MPT_E_INTERNAL, "%s: %s", where, e.what());
    } catch (...) {
        return fail(MPT_E_INTERNAL, "%s: unexpected exception", where);
    }
}

}  // namespace mptlib

#define MPT_HIP_TRY(expr)                                                                  \
    do {                                                                                   \
        hipError_t e_ = (expr);                                                            \
        if (e_ != hipSuccess)                                                              \
            return mptlib::fail(MPT_E_DEVICE, "%s: %s (%s:%d)", #expr, hipGetErrorString(e_), \
                                __FILE__, __LINE__);                                       \
    } while (0)
