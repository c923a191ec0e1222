#include "device_cache.h"

#include <atomic>
#include <cstdint>
#include <deque>
#include <map>
#include <mutex>
#include <unordered_map>
#include <vector>

namespace fmm {
namespace {

struct Idle {
    void *p;
    size_t bytes;
    int device;
};

struct Cache {
    std::mutex mu;
    std::unordered_map<void *, Idle> live;     // blocks handed out
    std::deque<Idle> idle;                     // oldest first
    std::map<int, size_t> idle_bytes;          // per device
    std::map<int, std::vector<SideStream>> streams;
};

// Never destroyed: trees may outlive static destruction order, and the runtime releases
// the device's memory at process exit.
Cache &cache()
{
    static Cache *c = new Cache();
    return *c;
}

// Sizes in steps of an eighth of the power of two below, so that slightly different trees
// can use each other's blocks.
size_t rounded(size_t bytes)
{
    size_t step = 256;
    while (step * 16 <= bytes) step *= 2;
    return (bytes + step - 1) / step * step;
}

// Returns everything held idle on the current device: the cache's blocks, and what the pool has
// taken back.
void release_idle()
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return;
    Cache &c = cache();
    std::vector<void *> drop;
    {
        std::lock_guard<std::mutex> lock(c.mu);
        std::deque<Idle> rest;
        for (const Idle &b : c.idle)
            if (b.device == dev) drop.push_back(b.p);
            else rest.push_back(b);
        c.idle.swap(rest);
        c.idle_bytes[dev] = 0;
    }
    for (void *q : drop) (void)hipFree(q);
    hipMemPool_t pool;
    if (hipDeviceGetDefaultMemPool(&pool, dev) == hipSuccess) (void)hipMemPoolTrimTo(pool, 0);
    (void)hipGetLastError();
}

template <typename Alloc> hipError_t again_without_idle(void **p, Alloc alloc)
{
    hipError_t e = alloc();
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        release_idle();
        e = alloc();
    }
    if (e != hipSuccess) {
        *p = nullptr;
        (void)hipGetLastError();
    }
    return e;
}

}  // namespace

hipError_t device_malloc(void **p, size_t bytes)
{
    return again_without_idle(p, [&] { return hipMalloc(p, bytes); });
}

hipError_t pool_malloc(void **p, size_t bytes, hipStream_t s)
{
    return again_without_idle(p, [&] { return hipMallocAsync(p, bytes, s); });
}

hipError_t block_alloc(void **p, size_t bytes)
{
    *p = nullptr;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const size_t want = rounded(bytes ? bytes : 1);
    Cache &c = cache();
    {
        std::lock_guard<std::mutex> lock(c.mu);
        auto best = c.idle.end();
        for (auto it = c.idle.begin(); it != c.idle.end(); ++it)
            if (it->device == dev && it->bytes >= want && it->bytes / 2 <= want &&
                (best == c.idle.end() || it->bytes < best->bytes))
                best = it;
        if (best != c.idle.end()) {
            const Idle b = *best;
            c.idle.erase(best);
            c.idle_bytes[dev] -= b.bytes;
            c.live.emplace(b.p, b);
            *p = b.p;
            return hipSuccess;
        }
    }
    e = device_malloc(p, want);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lock(c.mu);
    c.live.emplace(*p, Idle{*p, want, dev});
    return hipSuccess;
}

void block_free(void *p)
{
    if (!p) return;
    Cache &c = cache();
    std::vector<void *> drop;
    {
        std::lock_guard<std::mutex> lock(c.mu);
        auto it = c.live.find(p);
        if (it == c.live.end()) return;
        const Idle b = it->second;
        c.live.erase(it);
        c.idle.push_back(b);
        size_t &sum = c.idle_bytes[b.device];
        sum += b.bytes;
        for (auto k = c.idle.begin(); sum > kIdleBytes && k != c.idle.end();) {
            if (k->device != b.device) {
                ++k;
                continue;
            }
            sum -= k->bytes;
            drop.push_back(k->p);
            k = c.idle.erase(k);
        }
    }
    for (void *q : drop) (void)hipFree(q);
}

void retain_pool(int device)
{
    static std::atomic<uint64_t> done{0};
    if (device < 0 || device >= 64 || ((done.load() >> device) & 1)) return;
    hipMemPool_t pool;
    if (hipDeviceGetDefaultMemPool(&pool, device) == hipSuccess) {
        uint64_t threshold = UINT64_MAX;
        (void)hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &threshold);
    }
    (void)hipGetLastError();
    done.fetch_or(uint64_t(1) << device);
}

void bound_idle(int device)
{
    size_t idle;
    {
        Cache &c = cache();
        std::lock_guard<std::mutex> lock(c.mu);
        idle = c.idle_bytes[device];
    }
    const uint64_t rest = kIdleBytes > idle ? kIdleBytes - idle : 0;
    hipMemPool_t pool;
    uint64_t used = 0, reserved = 0;
    auto excess = [&]() {
        return hipMemPoolGetAttribute(pool, hipMemPoolAttrUsedMemCurrent, &used) == hipSuccess &&
               hipMemPoolGetAttribute(pool, hipMemPoolAttrReservedMemCurrent, &reserved) == hipSuccess &&
               reserved > used + rest;
    };
    if (hipDeviceGetDefaultMemPool(&pool, device) == hipSuccess && excess()) {
        (void)hipMemPoolTrimTo(pool, used + rest);
        if (excess()) (void)hipMemPoolTrimTo(pool, rest);
    }
    (void)hipGetLastError();
}

hipError_t side_stream_take(int device, SideStream &s)
{
    Cache &c = cache();
    {
        std::lock_guard<std::mutex> lock(c.mu);
        auto &v = c.streams[device];
        if (!v.empty()) {
            s = v.back();
            v.pop_back();
            return hipSuccess;
        }
    }
    s = SideStream{};
    hipError_t e = hipStreamCreateWithFlags(&s.stream, hipStreamNonBlocking);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&s.fork, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&s.join, hipEventDisableTiming);
    return e;
}

void side_stream_give(int device, SideStream &s)
{
    if (s.stream && s.fork && s.join) {
        Cache &c = cache();
        std::lock_guard<std::mutex> lock(c.mu);
        auto &v = c.streams[device];
        if (v.size() < kIdleStreams) {
            v.push_back(s);
            s = SideStream{};
            return;
        }
    }
    if (s.stream) hipStreamDestroy(s.stream);
    if (s.fork) hipEventDestroy(s.fork);
    if (s.join) hipEventDestroy(s.join);
    s = SideStream{};
}

}  // namespace fmm
