// Drives the staged host transfers on a host-side runtime (hip_host.h).
#include "hip_host.h"

#include "wcl_stage.cpp"

#include <cstdarg>

void wcl_set_error(const char*, ...) {}

// The copies are ordered on the caller's stream, whatever handle names it:
// what the caller has queued there before is done before them.
static int ordered(const char* name, hipStream_t st) {
    const size_t n = 5 * kChunk + 1000;   // six chunks, the last one ragged
    std::vector<char> dev(n, 'o'), out(n, '?'), seen(n, '?'), src(n, 's');
    host::enqueue(st, [&] { std::fill(dev.begin(), dev.end(), 'n'); });   // what an unpack writes
    HOST_CHECK(name, stage_to_host(0, out.data(), dev.data(), n, st) == WCL_OK);
    HOST_CHECK(name, out == std::vector<char>(n, 'n'));
    host::enqueue(st, [&] { seen = dev; });   // a pack that still reads the block
    HOST_CHECK(name, stage_to_device(0, dev.data(), src.data(), n, st) == WCL_OK);
    HOST_CHECK(name, hipStreamSynchronize(st) == hipSuccess);
    HOST_CHECK(name, seen == std::vector<char>(n, 'n'));
    HOST_CHECK(name, dev == src);
    // nothing went to the stream that the same handle names in another thread
    for (auto& kv : host::queues)
        HOST_CHECK(name, kv.first.first != hipStreamPerThread || kv.first.second == std::this_thread::get_id());
    std::printf("ok %s\n", name);
    return 0;
}

int main() {
    stage_ref();
    int own = 0;
    int rc = ordered("default-stream", nullptr) || ordered("own-stream", (hipStream_t)&own) ||
             ordered("per-thread-stream", hipStreamPerThread);
    stage_unref();
    return rc;
}
