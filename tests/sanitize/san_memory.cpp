// The block cache of released device memory (csrc/memory.cpp) over a device of 63.75 MiB that is made up here.
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <mutex>
#include <thread>
#include <vector>

#include "common.hpp"

static const size_t kDevice = (size_t(64) << 20) - (size_t(256) << 10);
static std::map<void *, size_t> live;
static std::mutex live_mutex;
static size_t in_use = 0, mallocs = 0;
static std::atomic<size_t> syncs{0};

extern "C" {
hipError_t hipMalloc(void **p, size_t bytes) {
    std::lock_guard<std::mutex> lock(live_mutex);
    ++mallocs;
    if (in_use + bytes > kDevice) return hipErrorOutOfMemory;
    *p = std::malloc(1);
    live[*p] = bytes;
    in_use += bytes;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    std::lock_guard<std::mutex> lock(live_mutex);
    if (!live.count(p)) std::abort();
    in_use -= live[p];
    live.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { ++syncs; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMemGetInfo(size_t *free_b, size_t *total_b) {
    *free_b = kDevice - in_use;
    *total_b = kDevice;
    return hipSuccess;
}
}

#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)

using namespace cst;

int main() {
    void *a = nullptr, *b = nullptr;
    const size_t MiB = size_t(1) << 20;
    {
        MemoryUser user;
        CHECK(device_alloc(&a, 20 * MiB + 100) == hipSuccess);
        CHECK(in_use <= 22 * MiB + 100);                        // rounded up by 2 MiB at most
        device_free(a);
        CHECK(syncs == 1 && in_use > 0);                        // kept while an object is alive ...
        size_t free_b = 0;
        CHECK(device_free_bytes(&free_b) == hipSuccess && free_b == kDevice);      // ... counts as free ...
        const size_t before = mallocs;
        CHECK(device_alloc(&b, 19 * MiB) == hipSuccess && b == a && mallocs == before);   // ... and reused
        CHECK(device_alloc(&a, 64) == hipSuccess);
        device_free(b);
        release_idle_memory();
        CHECK(live.size() == 1 && live.count(a) == 1);          // what is in use stays
        device_free(a);
        // what is kept does not stand in the way of a larger request, nor does the rounding: 63.5 MiB would be 64
        CHECK(device_alloc(&a, 63 * MiB + MiB / 2) == hipSuccess && live.size() == 1);
        CHECK(device_alloc(&b, 257 * 1024) == hipErrorOutOfMemory && b == nullptr);
        CHECK(device_alloc(&b, 250 * 1024) == hipSuccess);
        device_free(b);
        device_free(a);
    }
    CHECK(live.empty() && in_use == 0);                         // nothing is kept when the last object is gone
    {
        MemoryUser user;
        std::vector<std::thread> threads;
        for (int t = 0; t < 8; ++t)
            threads.emplace_back([t] {
                for (int i = 0; i < 2000; ++i) {
                    void *p = nullptr;
                    if (device_alloc(&p, size_t(1000 + (t * 7919 + i * 104729) % 500000)) == hipSuccess) device_free(p);
                }
            });
        for (auto &t : threads) t.join();
    }
    CHECK(live.empty() && in_use == 0);
    std::printf("san_memory: ok\n");
    return 0;
}
