// Large copies between pageable host memory and the device through pinned
// staging chunks, filled or emptied by a few host threads while the chunks
// before them cross PCIe.  One host thread's copy into the runtime's own
// staging is what bounds a plain hipMemcpy from pageable memory, and on the
// way back the page faults of a fresh destination, which one thread takes one
// after the other.
//
// The staging sets are shared by the contexts of the process: at most kSets of
// kThreads * 2 chunks (16 MiB) each, allocated on first use and freed with the
// last context.  A call that finds every set taken copies directly.
//
// Measured: pack + unpack of a 25 MB FP64 source (16^3x32) 2.94 -> 1.75 ms
// (0.47 ms each way at the pinned rate of 54 GB/s), the upload of 75 MB of
// links with the clover build and a D-apply 3.19 -> 2.33 ms (2.1 with the
// clover build of today and the device block kept).  Threads x chunk:
// 4 x 1 MiB 1.96 / 2.96 ms, 8 x 1 MiB 2.42 / 3.01, 4 x 2 MiB 1.74 / 2.48,
// 3 x 4 MiB 1.72 / 2.30, 2 x 4 MiB 1.75 / 2.33: each chunk's copy and event
// cost more than the overlap of smaller ones gains.
#include <algorithm>
#include <atomic>
#include <cstring>
#include <thread>
#include <vector>

#include "wcl_kernels.h"

namespace {

constexpr size_t kChunk = 4u << 20;
constexpr int kThreads = 2, kSets = 4;
constexpr size_t kMin = 8u << 20;   // smaller copies go directly: there is nothing to overlap

std::mutex g_mu;
std::vector<char*> g_free;
int g_live = 0, g_refs = 0;

void free_set(char* p) { (void)hipHostFree(p); }

char* take_set() {
    {
        std::lock_guard<std::mutex> lk(g_mu);
        if (!g_free.empty()) {
            char* p = g_free.back();
            g_free.pop_back();
            return p;
        }
        if (g_live == kSets) return nullptr;
        ++g_live;
    }
    void* p = nullptr;
    if (hipHostMalloc(&p, kThreads * 2 * kChunk, hipHostMallocPortable) == hipSuccess) return (char*)p;
    (void)hipGetLastError();
    std::lock_guard<std::mutex> lk(g_mu);
    --g_live;
    return nullptr;
}

void give_set(char* p) {
    {
        std::lock_guard<std::mutex> lk(g_mu);
        if (g_refs > 0) {
            g_free.push_back(p);   // room reserved in stage_ref
            return;
        }
        --g_live;
    }
    free_set(p);
}

// Memory the runtime already knows (pinned) is copied directly.
bool pageable(const void* p) {
    hipPointerAttribute_t at{};
    if (hipPointerGetAttributes(&at, p) != hipSuccess) {
        (void)hipGetLastError();
        return true;
    }
    return at.type == hipMemoryTypeUnregistered;
}

// Chunks t, t + T, ... of the copy, two staging slots.
template <bool TO_DEVICE>
hipError_t stripe(int device, char* dev, char* host, size_t bytes, hipStream_t st, char* slots, int t, int T) {
    hipError_t e = hipSetDevice(device);
    hipEvent_t ev[2] = {nullptr, nullptr};
    for (int s = 0; s < 2 && e == hipSuccess; ++s) e = hipEventCreateWithFlags(&ev[s], hipEventDisableTiming);
    const size_t n = (bytes + kChunk - 1) / kChunk;
    size_t held[2];          // chunk in each slot
    bool busy[2] = {false, false};
    auto size_of = [&](size_t c) { return std::min(kChunk, bytes - c * kChunk); };
    auto drain = [&](int s) {   // wait for slot s; on the way back, empty it
        if (!busy[s]) return;
        busy[s] = false;
        const hipError_t w = hipEventSynchronize(ev[s]);
        if (e == hipSuccess) e = w;
        if (!TO_DEVICE && e == hipSuccess) memcpy(host + held[s] * kChunk, slots + s * kChunk, size_of(held[s]));
    };
    int s = 0;
    for (size_t c = t; c < n && e == hipSuccess; c += T, s ^= 1) {
        char* slot = slots + s * kChunk;
        drain(s);
        if (e != hipSuccess) break;
        if (TO_DEVICE) memcpy(slot, host + c * kChunk, size_of(c));
        e = TO_DEVICE ? hipMemcpyAsync(dev + c * kChunk, slot, size_of(c), hipMemcpyHostToDevice, st)
                      : hipMemcpyAsync(slot, dev + c * kChunk, size_of(c), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipEventRecord(ev[s], st);
        if (e != hipSuccess) {
            (void)hipStreamSynchronize(st);   // nothing may still use the slot
            break;
        }
        busy[s] = true;
        held[s] = c;
    }
    drain(s);
    drain(s ^ 1);
    for (auto x : ev)
        if (x) (void)hipEventDestroy(x);
    return e;
}

template <bool TO_DEVICE>
int copy(int device, void* dev, void* host, size_t bytes, hipStream_t st) {
    char* set = bytes >= kMin && pageable(host) ? take_set() : nullptr;
    if (!set) {
        WCL_HIP(TO_DEVICE ? hipMemcpyAsync(dev, host, bytes, hipMemcpyHostToDevice, st)
                          : hipMemcpyAsync(host, dev, bytes, hipMemcpyDeviceToHost, st));
        if (!TO_DEVICE) WCL_HIP(hipStreamSynchronize(st));
        return WCL_OK;
    }
    // hipStreamPerThread names another stream in every thread: only the caller's
    // own is ordered with what it has queued there, so it does all the stripes
    const int T = st == hipStreamPerThread
                      ? 1
                      : std::max(1, std::min(kThreads, (int)std::thread::hardware_concurrency() / 2));
    hipError_t err[kThreads];
    std::fill(err, err + kThreads, hipSuccess);
    std::thread th[kThreads];
    auto work = [&](int t) {
        err[t] = stripe<TO_DEVICE>(device, (char*)dev, (char*)host, bytes, st, set + (size_t)t * 2 * kChunk, t, T);
    };
    bool started[kThreads] = {};
    for (int t = 1; t < T; ++t) {
        try {
            th[t] = std::thread(work, t);
            started[t] = true;
        } catch (...) {   // no thread: this one does that stripe too
        }
    }
    work(0);
    for (int t = 1; t < T; ++t) {
        if (started[t]) th[t].join();
        else work(t);
    }
    give_set(set);
    for (int t = 0; t < T; ++t) WCL_HIP(err[t]);
    return WCL_OK;
}

}  // namespace

void stage_ref() {
    std::lock_guard<std::mutex> lk(g_mu);
    ++g_refs;
    g_free.reserve(kSets);
}

void stage_unref() {
    std::vector<char*> gone;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        if (--g_refs > 0) return;
        gone.swap(g_free);
        g_live -= (int)gone.size();
    }
    for (char* p : gone) free_set(p);
}

int stage_to_device(int device, void* dev, const void* host, size_t bytes, hipStream_t st) {
    return copy<true>(device, dev, const_cast<void*>(host), bytes, st);
}

int stage_to_host(int device, void* host, const void* dev, size_t bytes, hipStream_t st) {
    return copy<false>(device, const_cast<void*>(dev), host, bytes, st);
}
