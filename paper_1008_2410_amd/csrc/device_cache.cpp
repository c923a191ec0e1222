#include "device_cache.h"

#include <atomic>
#include <cstdint>
#include <list>
#include <mutex>
#include <unordered_map>

namespace fmm {
namespace {

constexpr int kDevices = 64;

struct Block {
    void *p;
    size_t bytes;
    int device;
};

// A block keeps its list node and its place in `where` from the allocation to the release of its
// memory: giving blocks back, here and to the device, allocates no host memory and cannot throw.
struct Cache {
    std::mutex mu;
    std::list<Block> live;  // handed out
    std::list<Block> idle;  // oldest first
    std::unordered_map<void *, std::list<Block>::iterator> where;
    size_t idle_bytes[kDevices] = {};
    struct {
        SideStream s[kIdleStreams];
        size_t count = 0;
    } streams[kDevices];
};

// Never destroyed: trees may outlive static destruction order, and the runtime releases
// the device's memory at process exit.
Cache &cache()
{
    static Cache *c = new Cache();
    return *c;
}

// Takes the device's oldest idle blocks out of the cache until at most `keep` bytes are idle.
std::list<Block> take_oldest(Cache &c, int device, size_t keep)
{
    std::list<Block> out;
    for (auto k = c.idle.begin(); c.idle_bytes[device] > keep && k != c.idle.end();) {
        const auto next = std::next(k);
        if (k->device == device) {
            c.idle_bytes[device] -= k->bytes;
            c.where.erase(k->p);
            out.splice(out.end(), c.idle, k);
        }
        k = next;
    }
    return out;
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
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kDevices) return;
    Cache &c = cache();
    std::list<Block> drop;
    {
        std::lock_guard<std::mutex> lock(c.mu);
        drop = take_oldest(c, dev, 0);
    }
    for (const Block &b : drop) (void)hipFree(b.p);
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
    if (dev < 0 || dev >= kDevices) return hipErrorInvalidDevice;
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
            c.idle_bytes[dev] -= best->bytes;
            c.live.splice(c.live.end(), c.idle, best);
            *p = best->p;
            return hipSuccess;
        }
    }
    e = device_malloc(p, want);
    if (e != hipSuccess) return e;
    try {
        std::lock_guard<std::mutex> lock(c.mu);
        c.live.push_back(Block{*p, want, dev});
        try {
            c.where.emplace(*p, std::prev(c.live.end()));
        } catch (...) {
            c.live.pop_back();
            throw;
        }
    } catch (...) {  // no host memory for its entry
        (void)hipFree(*p);
        *p = nullptr;
        return hipErrorOutOfMemory;
    }
    return hipSuccess;
}

void block_free(void *p)
{
    if (!p) return;
    Cache &c = cache();
    std::list<Block> drop;
    {
        std::lock_guard<std::mutex> lock(c.mu);
        const auto it = c.where.find(p);
        if (it == c.where.end()) return;
        const auto b = it->second;
        c.idle.splice(c.idle.end(), c.live, b);
        c.idle_bytes[b->device] += b->bytes;
        drop = take_oldest(c, b->device, kIdleBytes);
    }
    for (const Block &b : drop) (void)hipFree(b.p);
}

void retain_pool(int device)
{
    static std::atomic<uint64_t> done{0};
    if (device < 0 || device >= kDevices || ((done.load() >> device) & 1)) return;
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
    if (device < 0 || device >= kDevices) return;
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
    if (device >= 0 && device < kDevices) {
        Cache &c = cache();
        std::lock_guard<std::mutex> lock(c.mu);
        auto &v = c.streams[device];
        if (v.count > 0) {
            s = v.s[--v.count];
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
    if (s.stream && s.fork && s.join && device >= 0 && device < kDevices) {
        Cache &c = cache();
        std::lock_guard<std::mutex> lock(c.mu);
        auto &v = c.streams[device];
        if (v.count < kIdleStreams) {
            v.s[v.count++] = s;
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
