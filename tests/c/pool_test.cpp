// The pool of pinned blocks under calls that fail, on the CPU: libmpt.so with
// this program's own stand-ins for the HIP calls it makes (the executable's
// symbols come first), so that a stream that is being captured, a stale error
// and a failing allocation can be played without a device. Kernels do not run;
// what is checked is which way the results would have come back: through a
// block (no copy is enqueued) or by a copy (the way without a block); and that a
// call which runs out of host memory returns an error.
// Exit status 0 when every check passed.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>

#include "mpt.h"

static bool no_memory = false;
void *operator new(size_t n) {
    void *p = no_memory ? nullptr : malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }

static bool capturing = false, device_lost = false;
static int stale = 0, copies = 0, allocations = 0;
static const hipError_t kRefused = hipErrorStreamCaptureUnsupported;

extern "C" {
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned) {
    ++allocations;
    *p = calloc(1, bytes);
    return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *) { return hipSuccess; }
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError(void) {
    const bool err = stale > 0;
    if (err) --stale;
    return err ? hipErrorInvalidValue : hipSuccess;
}
hipError_t hipMemcpyAsync(void *dst, const void *, size_t bytes, hipMemcpyKind kind, hipStream_t) {
    ++copies;
    if (kind == hipMemcpyDeviceToHost) memset(dst, 0, bytes);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
    return device_lost ? hipErrorUnknown : capturing ? kRefused : hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *st) {
    *st = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
}

static int failures = 0;
#define CHECK(cond)                                                                                           \
    do {                                                                                                      \
        if (!(cond)) {                                                                                        \
            fprintf(stderr, "FAIL line %d: %s (last error: %s)\n", __LINE__, #cond, mpt_last_error());        \
            ++failures;                                                                                       \
        }                                                                                                     \
    } while (0)

static char arrays[16][4096] __attribute__((aligned(256)));
static char workspace[1 << 20] __attribute__((aligned(256)));
// one call of each kind that takes a block; the number that returned MPT_OK
static int calls() {
    void *a = arrays[0], *b = arrays[1], *c = arrays[2];
    int64_t out = 0;
    int ok = 0;
    auto count = [&](int rc) { ok += rc == MPT_OK; };
    count(mpt_build_weights(4, 8, 8, (int64_t *)a, (int64_t *)b, (int32_t *)c, (uint32_t *)arrays[3],
                            (int64_t *)arrays[4], workspace, sizeof workspace, nullptr));
    count(mpt_solve_exact(4, (int64_t *)arrays[4], (int64_t *)arrays[5], (uint32_t *)arrays[6], &out, workspace,
                          sizeof workspace, nullptr));
    count(mpt_extract_orders(4, 8, 8, (int64_t *)b, (int32_t *)c, (uint32_t *)arrays[3], (uint32_t *)arrays[6],
                             (int32_t *)arrays[7], workspace, sizeof workspace, nullptr));
    count(mpt_spanning_tree_bound(2, (int64_t *)a, &out, workspace, sizeof workspace, nullptr));
    count(mpt_layout_cost(4, 8, 8, (int64_t *)a, (int64_t *)b, (int32_t *)c, nullptr, &out, workspace,
                          sizeof workspace, nullptr));
    return ok;
}
// all calls succeed, and every result came through a block
static bool through_blocks() {
    const int before = copies;
    return calls() == 5 && copies == before;
}

int main() {
    CHECK(through_blocks());
    // more refused calls than the pool has blocks
    capturing = true;
    for (int i = 0; i < 40; ++i) CHECK(calls() == 0);
    capturing = false;
    CHECK(through_blocks());
    // an error left by somebody's earlier call: these calls fail, later ones do not
    for (int i = 0; i < 40; ++i) {
        stale = 1 << 20;
        CHECK(calls() == 0);
        stale = 0;
    }
    CHECK(through_blocks());
    // a wait that fails for another reason: the device may still write the
    // block, so it stays away, and with all of them gone results are copied
    device_lost = true;
    for (int i = 0; i < 40; ++i) CHECK(calls() == 0);
    device_lost = false;
    const int before = copies;
    CHECK(calls() == 5 && copies == before + 5);
    CHECK(allocations == 1);
    // host memory that runs out inside a call is an error of that call: no C++
    // exception crosses the interface
    int64_t window = 2, capacity = 5, cost = 0;
    no_memory = true;
    const int rc = mpt_cache_simulate(4, 8, 8, (int64_t *)arrays[0], (int64_t *)arrays[1], (int32_t *)arrays[2], 1,
                                      &window, &capacity, &cost, nullptr, workspace, sizeof workspace, nullptr);
    no_memory = false;
    CHECK(rc == MPT_E_INTERNAL);
    CHECK(strstr(mpt_last_error(), "mpt_cache_simulate") != nullptr);
    if (!failures) puts("all checks hold");
    return failures ? 1 : 0;
}
