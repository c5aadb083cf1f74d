// The host transfers of the library run on the CPU against a stand-in for the
// HIP runtime, which records who queues what.  Prints one line per fault and
// "done"; tests/test_transfer_host.py compiles and runs it.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <set>
#include <string>
#include <thread>
#include <vector>

#include "fs_runtime.hpp"

namespace {

std::mutex mu;
std::set<std::thread::id> queued_by;  // threads that queued copies, events or kernels
std::atomic<int> fail_events{0};      // hipEventRecord calls that fail from now on
std::atomic<int> unwaited{0};         // 1: a kernel writes a pinned buffer and nobody has waited for it
int given_unwaited = 0;               // buffers taken or freed meanwhile

void queued()
{
    std::lock_guard<std::mutex> lk(mu);
    queued_by.insert(std::this_thread::get_id());
}

} // namespace

namespace fsr {
thread_local std::string g_err;
fs_status fail(fs_status s, const std::string& m)
{
    g_err = m;
    return s;
}
} // namespace fsr

extern "C" {
hipError_t hipHostMalloc(void** p, size_t n, unsigned)
{
    *p = std::malloc(n);
    return hipSuccess;
}
hipError_t hipHostFree(void* p)
{
    given_unwaited += unwaited;
    std::free(p);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned)
{
    *e = (hipEvent_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e)
{
    std::free((void*)e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t)
{
    queued();
    if (fail_events > 0) {
        --fail_events;
        return hipErrorUnknown;
    }
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t)
{
    unwaited = 0;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t)
{
    unwaited = 0;
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t)
{
    queued();
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t)
{
    queued();
    unwaited = 1; // (the kernel's arrays are not filled: only the order is looked at)
    return hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* m, hipStream_t* s)
{
    *g = *b = dim3(1);
    *m = 0;
    *s = nullptr;
    return hipSuccess;
}
void** __hipRegisterFatBinary(const void*) { return nullptr; }
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipUnregisterFatBinary(void**) {}
char __hip_fatbin[8];
}

int main()
{
    const size_t n = 3 * ((size_t)1 << 17) + 7;
    std::vector<int32_t> state(n), back(n, -1);
    std::vector<float> age(n), age_back(n, -1.0f);
    for (size_t i = 0; i < n; ++i) {
        state[i] = (int32_t)(i % 4);
        age[i] = (float)i;
    }
    std::vector<uint8_t> d_state(n);
    std::vector<float> d_age(n);
    fsr::graph_opened();
    // a round trip on a stream of its own may use several threads; on the
    // per-thread stream every thread's handle names another stream, so the
    // caller's thread alone may queue work
    for (hipStream_t s : {(hipStream_t)&mu, hipStreamPerThread}) {
        queued_by.clear();
        bool bad_state = true, bad_age = true;
        if (fsr::copy_in(0, s, n, state.data(), d_state.data(), age.data(), d_age.data(), 4, true, &bad_state, &bad_age) !=
                FS_OK || bad_state || bad_age)
            std::puts("copy_in failed");
        if (fsr::copy_out(0, s, n, d_state.data(), back.data(), d_age.data(), age_back.data(), 4) != FS_OK)
            std::puts("copy_out failed");
        if (back != state || age_back != age) std::puts("round trip differs");
        if (s == hipStreamPerThread && (queued_by.size() != 1 || *queued_by.begin() != std::this_thread::get_id()))
            std::puts("per-thread stream: work queued by other threads");
        std::fill(back.begin(), back.end(), -1);
    }
    // a read whose event cannot be recorded waits for its kernel before the
    // pinned buffer goes back to the pool or is freed
    for (bool keep : {true, false}) {
        if (!keep) fsr::graph_closed(); // (no graph is open: buffers are freed, not kept)
        fail_events = 1;
        int64_t rows[4 * 3];
        if (fsr::copy_history(0, (hipStream_t)&mu, nullptr, 1, 0, 0, 8, 3, rows) == FS_OK) std::puts("error lost");
        given_unwaited += unwaited; // (the buffer is free for the next taker now)
        unwaited = 0;
    }
    if (given_unwaited) std::puts("buffer given up under a running kernel");
    std::puts("done");
    return 0;
}
