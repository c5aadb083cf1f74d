// Per-node arrays between the caller's host arrays and device memory.
//
// A state load or read moves 5 to 9 bytes per node through host memory, and
// the caller's arrays are usually fresh pages; one pageable copy on one core,
// with the reordering of a degree-sorted graph done by that core, took 3.7 ms
// per load and read of 1e6 nodes (a 500-step solve takes 7.3).  Here the device
// reorders and narrows states to bytes, and the arrays go in pieces through
// pinned buffers, each piece copied, widened or checked by one of a few
// threads while the next pieces are on their way.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstring>
#include <exception>
#include <functional>
#include <mutex>
#include <thread>
#include <vector>

#include "fs_runtime.hpp"

namespace fsr {

namespace {

// Nodes per piece, and the most threads (and so pinned buffers) of one call.
constexpr size_t PIECE = (size_t)1 << 17;
constexpr size_t MAX_THREADS = 8;
// A pinned buffer holds a piece's states (one byte each) after its payload
// (up to four bytes each).
constexpr size_t SLOT_BYTES = PIECE * 5;

struct Slot {
    int device = -1;
    char* host = nullptr;
    hipEvent_t ev = nullptr;
};

void destroy(Slot& s)
{
    if (s.ev) (void)hipEventDestroy(s.ev);
    if (s.host) (void)hipHostFree(s.host);
    s = Slot{};
}

// Idle pinned buffers of all devices: at most 2 MAX_THREADS are kept (10 MiB),
// more are made and freed by the calls that need them.  They go when the last
// graph is released.
std::mutex g_mu;
std::vector<Slot> g_idle;
size_t g_graphs = 0;

hipError_t take(int device, Slot& out)
{
    {
        std::lock_guard<std::mutex> lk(g_mu);
        for (size_t i = 0; i < g_idle.size(); ++i)
            if (g_idle[i].device == device) {
                out = g_idle[i];
                g_idle.erase(g_idle.begin() + (long)i);
                return hipSuccess;
            }
    }
    Slot s;
    s.device = device;
    hipError_t e = hipHostMalloc((void**)&s.host, SLOT_BYTES, hipHostMallocDefault);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&s.ev, hipEventDisableTiming);
    if (e != hipSuccess) {
        destroy(s);
        return e;
    }
    out = s;
    return hipSuccess;
}

void give(Slot& s)
{
    if (!s.host) return;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        if (g_graphs > 0 && g_idle.size() < 2 * MAX_THREADS) {
            g_idle.push_back(s); // (capacity reserved by graph_opened)
            return;
        }
    }
    destroy(s);
}

// Runs f(first node, nodes, slot) for every piece of n nodes, on as many
// threads as there are pieces (up to MAX_THREADS), each with a pinned buffer of
// its own on `device`.  f returns a HIP error, which ends the run.  The handle
// hipStreamPerThread names another stream on every thread, so there the
// caller's thread, which has queued what the pieces wait for, takes them all.
template <class F>
fs_status for_pieces(int device, hipStream_t stream, size_t n, F f)
{
    const size_t pieces = (n + PIECE - 1) / PIECE;
    std::atomic<size_t> next{0};
    std::atomic<int> err{(int)hipSuccess};
    auto work = [&]() noexcept {
        Slot s;
        hipError_t e = hipSuccess;
        size_t p = next.fetch_add(1);
        if (p < pieces) e = take(device, s);
        for (; p < pieces && e == hipSuccess && err.load() == (int)hipSuccess; p = next.fetch_add(1))
            e = f(p * PIECE, std::min(PIECE, n - p * PIECE), s);
        // (a failed piece may have left a copy under way in the buffer)
        if (e != hipSuccess && s.host) (void)hipStreamSynchronize(stream);
        give(s);
        int ok = (int)hipSuccess;
        if (e != hipSuccess) err.compare_exchange_strong(ok, (int)e);
    };
    std::vector<std::thread> threads;
    const size_t most = stream == hipStreamPerThread ? 1 : MAX_THREADS;
    const size_t extra = std::min(pieces, most) - (pieces ? 1 : 0);
    try {
        threads.reserve(extra);
        for (size_t i = 0; i < extra; ++i)
            threads.emplace_back([&]() noexcept {
                if (hipSetDevice(device) == hipSuccess) work();
            });
    } catch (const std::exception&) {
        // fewer threads: the others take their pieces
    }
    work();
    for (std::thread& t : threads) t.join();
    const hipError_t e = (hipError_t)err.load();
    if (e != hipSuccess)
        return fail(e == hipErrorOutOfMemory ? FS_ERR_OUT_OF_MEMORY : FS_ERR_DEVICE,
                    std::string("host transfer: ") + hipGetErrorString(e));
    return FS_OK;
}

} // namespace

void graph_opened()
{
    std::lock_guard<std::mutex> lk(g_mu);
    g_idle.reserve(2 * MAX_THREADS);
    ++g_graphs;
}

void graph_closed()
{
    std::vector<Slot> drop;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        if (--g_graphs == 0) drop.swap(g_idle);
    }
    for (Slot& s : drop) destroy(s);
}

bool reads_direct(const fs_graph* g) { return g->h_orig.empty() && (size_t)g->n <= PIECE; }

fs_status read_direct(int device, hipStream_t stream, size_t n, size_t pay_bytes,
                      const std::function<hipError_t(uint8_t*, void*)>& put, int32_t* state, void* pay)
{
    Slot s;
    FS_HIP(take(device, s));
    uint8_t* st = (uint8_t*)s.host + PIECE * 4;
    hipError_t e = put(st, s.host);
    if (e == hipSuccess) e = hipEventRecord(s.ev, stream);
    if (e == hipSuccess) e = hipEventSynchronize(s.ev);
    if (e == hipSuccess) {
        std::memcpy(pay, s.host, n * pay_bytes);
        if (state)
            for (size_t i = 0; i < n; ++i) state[i] = st[i];
    } else {
        (void)hipStreamSynchronize(stream);
    }
    give(s);
    FS_HIP(e);
    return FS_OK;
}

fs_status copy_out(int device, hipStream_t stream, size_t n, const uint8_t* d_state, int32_t* state, const void* d_pay,
                   void* pay, size_t pay_bytes)
{
    return for_pieces(device, stream, n, [&](size_t at, size_t m, Slot& s) {
        // (arrays of one piece that lie end to end come in one copy)
        const bool joined = m == n && pay && state && d_state == (const uint8_t*)d_pay + n * pay_bytes;
        uint8_t* st = (uint8_t*)s.host + (joined ? n * pay_bytes : PIECE * 4);
        hipError_t e = hipSuccess;
        if (joined)
            e = hipMemcpyAsync(s.host, d_pay, n * (pay_bytes + 1), hipMemcpyDeviceToHost, stream);
        else if (pay)
            e = hipMemcpyAsync(s.host, (const char*)d_pay + at * pay_bytes, m * pay_bytes, hipMemcpyDeviceToHost, stream);
        if (e == hipSuccess && state && !joined) e = hipMemcpyAsync(st, d_state + at, m, hipMemcpyDeviceToHost, stream);
        if (e == hipSuccess) e = hipEventRecord(s.ev, stream);
        if (e == hipSuccess) e = hipEventSynchronize(s.ev);
        if (e != hipSuccess) return e;
        if (pay) std::memcpy((char*)pay + at * pay_bytes, s.host, m * pay_bytes);
        if (state) {
            int32_t* out = state + at;
            for (size_t i = 0; i < m; ++i) out[i] = st[i];
        }
        return e;
    });
}

fs_status copy_in(int device, hipStream_t stream, size_t n, const int32_t* state, uint8_t* d_state, const void* pay,
                  void* d_pay, size_t pay_bytes, bool float_ages, bool* bad_state, bool* bad_age)
{
    std::atomic<bool> wrong_state{false}, wrong_age{false};
    const fs_status st = for_pieces(device, stream, n, [&](size_t at, size_t m, Slot& s) {
        uint8_t* narrow = (uint8_t*)s.host + PIECE * 4;
        uint32_t any = 0;
        const int32_t* in = state + at;
        for (size_t i = 0; i < m; ++i) {
            any |= (uint32_t)in[i];
            narrow[i] = (uint8_t)in[i];
        }
        if (any > 3u) wrong_state = true;
        if (pay) {
            std::memcpy(s.host, (const char*)pay + at * pay_bytes, m * pay_bytes);
            if (float_ages) {
                // finite and >= 0: below the bits of infinity, or -0
                const uint32_t* w = (const uint32_t*)s.host;
                uint32_t bad = 0;
                for (size_t i = 0; i < m; ++i) bad |= (uint32_t)(w[i] >= 0x7F800000u) & (uint32_t)(w[i] != 0x80000000u);
                if (bad) wrong_age = true;
            }
        }
        hipError_t e = hipSuccess;
        if (wrong_state || wrong_age) return e; // (every piece is still checked)
        if (pay)
            e = hipMemcpyAsync((char*)d_pay + at * pay_bytes, s.host, m * pay_bytes, hipMemcpyHostToDevice, stream);
        if (e == hipSuccess) e = hipMemcpyAsync(d_state + at, narrow, m, hipMemcpyHostToDevice, stream);
        if (e == hipSuccess) e = hipEventRecord(s.ev, stream);
        if (e == hipSuccess) e = hipEventSynchronize(s.ev);
        return e;
    });
    *bad_state = wrong_state;
    *bad_age = wrong_age;
    return st;
}

// The counts of one replica in ring rows (first + i) mod H, i < n.
__global__ void history_rows_kernel(const uint4* __restrict__ hist, uint32_t R, uint32_t replica, uint32_t first,
                                    uint32_t H, uint32_t n, uint4* __restrict__ out)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = hist[(size_t)((first + i) % H) * R + replica];
}

fs_status copy_history(int device, hipStream_t stream, const uint32_t* d_hist, uint32_t R, uint32_t replica,
                       uint64_t first_step, uint32_t H, size_t n, int64_t* out)
{
    constexpr size_t ROWS = SLOT_BYTES / sizeof(uint4);
    Slot s;
    FS_HIP(take(device, s));
    hipError_t e = hipSuccess;
    for (size_t at = 0; at < n && e == hipSuccess; at += ROWS) {
        const uint32_t m = (uint32_t)std::min(ROWS, n - at);
        // (the rows are written straight into the pinned buffer)
        hipLaunchKernelGGL(history_rows_kernel, dim3((m + 255) / 256), dim3(256), 0, stream, (const uint4*)d_hist, R,
                           replica, (uint32_t)((first_step + at) % H), H, m, (uint4*)s.host);
        e = hipGetLastError();
        if (e == hipSuccess) e = hipEventRecord(s.ev, stream);
        if (e == hipSuccess) e = hipEventSynchronize(s.ev);
        if (e != hipSuccess) break;
        const uint32_t* h = (const uint32_t*)s.host;
        for (size_t j = 0; j < 4 * (size_t)m; ++j) out[4 * at + j] = (int64_t)h[j];
    }
    // (a failed wait may have left the kernel writing the buffer)
    if (e != hipSuccess) (void)hipStreamSynchronize(stream);
    give(s);
    FS_HIP(e);
    return FS_OK;
}

} // namespace fsr
