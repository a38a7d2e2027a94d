// A host-side stand-in for the few HIP runtime calls that the library's host
// code makes, so that its ordering and its memory accounting can be checked
// without a device.  "Device" memory is host memory.  A stream is a queue whose
// work runs only when something waits for it, so a result that depends on work
// of another stream, or of a stream nobody waited for, comes out wrong here
// every time.  hipStreamPerThread names one queue per calling thread.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <mutex>
#include <thread>
#include <utility>
#include <vector>

#define __align__(n) __attribute__((aligned(n)))
#define HIP_SYMBOL(x) x

namespace host {

using Key = std::pair<hipStream_t, std::thread::id>;
struct Queue {
    std::vector<std::function<void()>> work;
    size_t done = 0;
};
struct Event {
    Queue* q = nullptr;
    size_t upto = 0;
};

inline std::mutex mu;
inline std::map<Key, Queue> queues;
inline std::map<const char*, size_t> pinned;   // pinned buffers
inline size_t free_bytes = (size_t)-1;       // what hipMalloc still gives out
inline std::map<void*, size_t> blocks;       // live device blocks
inline std::vector<std::pair<void*, size_t>> cache;   // freed blocks: the same size comes back at the same address

inline Queue& queue(hipStream_t st) {
    const bool own = st == hipStreamPerThread;
    return queues[Key{st, own ? std::this_thread::get_id() : std::thread::id()}];
}
inline bool is_pinned(const void* p) {   // called with mu held
    auto it = pinned.upper_bound((const char*)p);
    if (it == pinned.begin()) return false;
    --it;
    return (const char*)p < it->first + it->second;
}
inline void run(Queue& q, size_t upto) {
    for (; q.done < upto; ++q.done) q.work[q.done]();
}
// a "kernel" on st
inline void enqueue(hipStream_t st, std::function<void()> f) {
    std::lock_guard<std::mutex> g(mu);
    queue(st).work.push_back(std::move(f));
}

}  // namespace host

extern "C" {

const char* hipGetErrorString(hipError_t) { return "host"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }

hipError_t hipMalloc(void** p, size_t n) {
    std::lock_guard<std::mutex> g(host::mu);
    if (n > host::free_bytes) return hipErrorOutOfMemory;
    *p = nullptr;
    for (size_t k = 0; k < host::cache.size(); ++k)
        if (host::cache[k].second == n) {
            *p = host::cache[k].first;
            host::cache.erase(host::cache.begin() + (long)k);
            break;
        }
    if (!*p) *p = std::malloc(n);
    host::free_bytes -= n;
    host::blocks[*p] = n;
    return hipSuccess;
}
// as the runtime does: waits for everything first
hipError_t hipFree(void* p) {
    std::lock_guard<std::mutex> g(host::mu);
    for (auto& kv : host::queues) host::run(kv.second, kv.second.work.size());
    host::free_bytes += host::blocks[p];
    host::cache.push_back({p, host::blocks[p]});
    host::blocks.erase(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    *p = std::malloc(n);
    std::lock_guard<std::mutex> g(host::mu);
    host::pinned[(const char*)*p] = n;
    return hipSuccess;
}
hipError_t hipHostFree(void* p) {
    std::lock_guard<std::mutex> g(host::mu);
    host::pinned.erase((const char*)p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
    std::lock_guard<std::mutex> g(host::mu);
    a->type = host::is_pinned(p) ? hipMemoryTypeHost : hipMemoryTypeUnregistered;
    return hipSuccess;
}

hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    *e = (hipEvent_t) new host::Event;
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
    delete (host::Event*)e;
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t st) {
    std::lock_guard<std::mutex> g(host::mu);
    host::Queue& q = host::queue(st);
    *(host::Event*)e = host::Event{&q, q.work.size()};
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
    std::lock_guard<std::mutex> g(host::mu);
    auto* ev = (host::Event*)e;
    if (ev->q) host::run(*ev->q, ev->upto);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t st) {
    std::lock_guard<std::mutex> g(host::mu);
    host::Queue& q = host::queue(st);
    host::run(q, q.work.size());
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() {
    std::lock_guard<std::mutex> g(host::mu);
    for (auto& kv : host::queues) host::run(kv.second, kv.second.work.size());
    return hipSuccess;
}
// a pageable source is read before the call returns
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind kind, hipStream_t st) {
    std::lock_guard<std::mutex> g(host::mu);
    host::Queue& q = host::queue(st);
    if (kind == hipMemcpyHostToDevice && !host::is_pinned(s)) {
        auto copy = std::vector<char>((const char*)s, (const char*)s + n);
        q.work.push_back([=] { std::memcpy(d, copy.data(), n); });
        return hipSuccess;
    }
    q.work.push_back([=] { std::memcpy(d, s, n); });
    return hipSuccess;
}

}  // extern "C"

#define HOST_CHECK(name, cond)                                            \
    do {                                                                  \
        if (!(cond)) {                                                    \
            std::printf("FAILED %s: %s (line %d)\n", name, #cond, __LINE__); \
            std::fflush(stdout);                                          \
            return 1;                                                     \
        }                                                                 \
    } while (0)
