// Device memory of the library's objects: a bounded cache of released blocks.
//
// A CSF build of 76 M nonzeros takes 2.5 GB of temporaries and hands out 1.2 GB of level arrays.  hipMalloc and
// hipFree of these cost 1 ms by themselves, but memory that goes back to the driver is cleared before it is
// handed out again, and a program that builds tensor after tensor outruns that: 45 to 90 ms per build where the
// kernels take 7.  Blocks of destroyed objects are therefore kept and reused, under these rules:
//   - at most kCachedBytes are kept; the block unused for longest goes first;
//   - when no CSF and no plan is alive, everything goes back to the driver, and so it does when an allocation
//     fails, before it is tried again, in the end with no rounding;
//   - conststn_release_memory gives them back at once, for programs whose other allocators need the room;
//   - releasing a block waits for the device, as hipFree does, so a block never reaches its next owner while
//     work on any stream may still touch it;
//   - one mutex guards the lists: any thread may allocate and release.
#include <algorithm>
#include <list>
#include <mutex>
#include <new>
#include <unordered_map>

#include "common.hpp"

namespace cst {

namespace {

constexpr size_t kCachedBytes = size_t(8) << 30;

struct Block { void *p; size_t bytes; int device; };

struct Cache {
    std::mutex m;
    std::list<Block> idle;                             // longest unused first
    std::unordered_map<void *, Block> used;
    size_t idle_bytes = 0;
    int64_t users = 0;
};

// never destroyed: objects may be released by other static destructors, and the process's end frees everything
Cache &cache() {
    static Cache *c = new Cache;
    return *c;
}

// Sizes are rounded up to an eighth of their leading power of two (256 bytes at least, 2 MiB at most), so that
// tensors of about the same size share blocks; an idle block serves a request that is up to an eighth smaller.
size_t up_to(size_t bytes, size_t step) { return (bytes + step - 1) / step * step; }
size_t rounded(size_t bytes) {
    size_t step = 256;
    while (step * 16 <= bytes && step < (size_t(2) << 20)) step *= 2;
    return up_to(bytes, step);
}

void give_back(Cache &c, size_t keep) {
    while (c.idle_bytes > keep) {
        const Block b = c.idle.front();
        c.idle.pop_front();
        c.idle_bytes -= b.bytes;
        (void)hipFree(b.p);
    }
}

}  // namespace

hipError_t device_alloc(void **p, size_t bytes) {
    *p = nullptr;
    int device = 0;
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return e;
    const size_t want = rounded(bytes);
    Cache &c = cache();
    std::lock_guard<std::mutex> lock(c.m);
    auto best = c.idle.end();
    for (auto it = c.idle.begin(); it != c.idle.end(); ++it)
        if (it->device == device && it->bytes >= want && it->bytes <= want + want / 8 &&
            (best == c.idle.end() || it->bytes < best->bytes))
            best = it;
    if (best != c.idle.end()) {
        try {
            c.used[best->p] = *best;
        } catch (const std::bad_alloc &) {
            return hipErrorOutOfMemory;
        }
        *p = best->p;
        c.idle_bytes -= best->bytes;
        c.idle.erase(best);
        return hipSuccess;
    }
    size_t got = want;
    e = hipMalloc(p, got);
    if (e != hipSuccess && !c.idle.empty()) {
        (void)hipGetLastError();
        give_back(c, 0);
        e = hipMalloc(p, got);
    }
    if (e != hipSuccess && up_to(bytes, 256) < want) {
        (void)hipGetLastError();
        got = up_to(bytes, 256);
        e = hipMalloc(p, got);
    }
    if (e != hipSuccess) {
        *p = nullptr;
        return e;
    }
    try {
        c.used[*p] = Block{*p, got, device};
    } catch (const std::bad_alloc &) {
        (void)hipFree(*p);
        *p = nullptr;
        return hipErrorOutOfMemory;
    }
    return hipSuccess;
}

hipError_t device_free_bytes(size_t *bytes) {
    size_t free_b = 0, total_b = 0;
    int device = 0;
    hipError_t e = hipGetDevice(&device);
    if (e == hipSuccess) e = hipMemGetInfo(&free_b, &total_b);
    if (e != hipSuccess) return e;
    Cache &c = cache();
    std::lock_guard<std::mutex> lock(c.m);
    for (const Block &b : c.idle)
        if (b.device == device) free_b += b.bytes;
    *bytes = free_b;
    return hipSuccess;
}

void device_free(void *p) {
    if (!p) return;
    Cache &c = cache();
    Block b;
    {
        std::lock_guard<std::mutex> lock(c.m);
        const auto it = c.used.find(p);
        if (it == c.used.end()) return;
        b = it->second;
        c.used.erase(it);
    }
    int device = 0;
    (void)hipGetDevice(&device);
    if (device != b.device) (void)hipSetDevice(b.device);
    const hipError_t e = hipDeviceSynchronize();
    if (device != b.device) (void)hipSetDevice(device);
    std::lock_guard<std::mutex> lock(c.m);
    if (e != hipSuccess || c.users == 0) {
        (void)hipFree(p);
        return;
    }
    try {
        c.idle.push_back(b);
    } catch (const std::bad_alloc &) {
        (void)hipFree(p);
        return;
    }
    c.idle_bytes += b.bytes;
    give_back(c, kCachedBytes);
}

void release_idle_memory() {
    Cache &c = cache();
    std::lock_guard<std::mutex> lock(c.m);
    give_back(c, 0);
}

MemoryUser::MemoryUser() {
    Cache &c = cache();
    std::lock_guard<std::mutex> lock(c.m);
    ++c.users;
}

MemoryUser::~MemoryUser() {
    Cache &c = cache();
    std::lock_guard<std::mutex> lock(c.m);
    if (--c.users == 0) give_back(c, 0);
}

}  // namespace cst
