// Building blocks shared by the device tree builds (tree_build.hip for the uniform tree,
// adaptive_build.hip for the adaptive one): stream-ordered temporaries, an error status,
// a device-wide exclusive scan, a stable radix sort and the bounding square.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <string>
#include <utility>
#include <vector>

#include "../../include/fmm2d.h"
#include "cost_order.h"
#include "device_cache.h"

namespace fmm {

inline unsigned grid_for(int64_t n, int per) { return (unsigned)std::max<int64_t>(1, (n + per - 1) / per); }

// A region of device memory that is idle during a build (the per-call region of the
// evaluation workspace that a rebuilt tree takes over), lent to the build's temporaries
// as a stack: a block is taken at the top and the top moves back down when the topmost
// blocks have been given back.  All of a build's work runs on one stream, so a block
// given back while kernels that use it are still queued is only reused by kernels queued
// after them.  Requests that do not fit go to the library's block cache.
struct BuildArena {
    char *base = nullptr;
    size_t cap = 0;
    struct Block {
        size_t off, end;
        bool live;
    };
    std::vector<Block> stack;
    void *take(size_t bytes)
    {
        const size_t off = stack.empty() ? 0 : (stack.back().end + 255) / 256 * 256;
        if (!base || off + bytes > cap) return nullptr;
        stack.push_back({off, off + bytes, true});
        return base + off;
    }
    void give(void *p)
    {
        for (Block &b : stack)
            if (base + b.off == (char *)p) b.live = false;
        while (!stack.empty() && !stack.back().live) stack.pop_back();
    }
};

// The arena of the build running on this host thread (null: temporaries from the cache).
inline thread_local BuildArena *t_build_arena = nullptr;

struct BuildArenaScope {
    BuildArena *prev;
    explicit BuildArenaScope(BuildArena *a) : prev(t_build_arena) { t_build_arena = a; }
    ~BuildArenaScope() { t_build_arena = prev; }
};

// The device memory of a build on stream s (one per build, the outermost counts): blocks
// its steps give back are taken again by its later steps in stream order, and enter the
// library's cache at its end, after the stream has been synchronised.
struct BuildScope;
inline thread_local BuildScope *t_build_scope = nullptr;
struct BuildScope {
    hipStream_t s;
    BuildScope *prev;
    std::vector<std::pair<void *, size_t>> freed;
    explicit BuildScope(hipStream_t stream) : s(stream), prev(t_build_scope)
    {
        if (!prev || prev->s != s) t_build_scope = this;
    }
    ~BuildScope()
    {
        if (t_build_scope != this) return;
        t_build_scope = prev;
        (void)hipStreamSynchronize(s);
        for (auto &f : freed) block_free(f.first);
    }
    BuildScope(const BuildScope &) = delete;
    BuildScope &operator=(const BuildScope &) = delete;
};

inline hipError_t build_alloc(void **p, size_t bytes, hipStream_t s)
{
    if (t_build_scope && t_build_scope->s == s) {
        auto &f = t_build_scope->freed;
        size_t best = f.size();
        for (size_t k = 0; k < f.size(); ++k)
            if (f[k].second >= bytes && f[k].second / 4 <= bytes && (best == f.size() || f[k].second < f[best].second))
                best = k;
        if (best < f.size()) {
            *p = f[best].first;
            f.erase(f.begin() + (long)best);
            return hipSuccess;
        }
    }
    return block_alloc(p, bytes);
}
inline void build_free(void *p, size_t bytes, hipStream_t s)
{
    if (!p) return;
    if (t_build_scope && t_build_scope->s == s) {
        try {
            t_build_scope->freed.emplace_back(p, bytes);
            return;
        } catch (...) {  // (called from destructors) no host memory: given back at once
        }
    }
    (void)hipStreamSynchronize(s);
    block_free(p);
}

// Device buffer owned for the duration of a build step.
template <typename T>
struct Buf {
    // given back in the order of the build's stream, so a temporary can be released while
    // kernels that use it are still queued
    T *p = nullptr;
    size_t bytes = 0;
    hipStream_t s = nullptr;
    BuildArena *arena = nullptr;  // the block came from this arena
    bool kept = false;
    Buf() = default;
    Buf(const Buf &) = delete;
    Buf &operator=(const Buf &) = delete;
    ~Buf()
    {
        if (!p) return;
        if (arena) arena->give(p);
        else build_free(p, bytes, s);
    }
    // keep: the buffer outlives the build (handed to the tree by release(), which gives it
    // back with block_free), so it never comes from the arena
    hipError_t alloc(int64_t count, hipStream_t stream, bool keep = false)
    {
        s = stream;
        kept = keep;
        bytes = (size_t)std::max<int64_t>(count, 1) * sizeof(T);
        if (!kept && t_build_arena) {
            if (void *q = t_build_arena->take(bytes)) {
                p = (T *)q;
                arena = t_build_arena;
                return hipSuccess;
            }
        }
        return build_alloc((void **)&p, bytes, stream);
    }
    // hands the buffer over (allocated with keep = true)
    T *release()
    {
        T *q = p;
        p = nullptr;
        return q;
    }
    void swap(Buf &o)
    {
        std::swap(p, o.p);
        std::swap(bytes, o.bytes);
        std::swap(s, o.s);
        std::swap(arena, o.arena);
        std::swap(kept, o.kept);
    }
};

struct Status {
    int code = FMM_OK;
    std::string msg;
    bool check(hipError_t e, const char *what)
    {
        if (e == hipSuccess) return true;
        if (code == FMM_OK) {
            code = e == hipErrorOutOfMemory ? FMM_ENOMEM : FMM_EDEVICE;
            msg = std::string(what) + ": " + hipGetErrorString(e);
        }
        return false;
    }
};

// Exclusive scan of n uint32 (totals below 2^32; in place allowed) on stream s;
// *total_host receives the sum (after a synchronisation of s) if non-null.
bool scan_exclusive(const uint32_t *in, uint32_t *out, int64_t n, uint32_t *total_host, hipStream_t s, Status &st);

// Stable LSD sort of (keys, vals) by the low `bits` bits of the keys, 8-bit digits; the
// result is in keys and vals (whose buffers may be swapped with the sort's own).
bool radix_sort(Buf<uint64_t> &keys, Buf<uint32_t> &vals, int64_t n, int bits, hipStream_t s, Status &st);

// The sums of v[0..NV) over a workgroup of 256 threads (all of them), added to dst by one thread
// each: an atomic per wavefront and value had every wavefront of the launch wait in line for the
// same few addresses (2^20 particles at depth 8: 28 us for three sums over 65536 leaves).
template <int NV>
__device__ __forceinline__ void block_add(unsigned long long *dst, const unsigned long long (&v)[NV])
{
    __shared__ unsigned long long part[4][NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        unsigned long long x = v[q];
        for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o);
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6][q] = x;
    }
    __syncthreads();
    if (threadIdx.x < NV) {
        const unsigned long long x =
            part[0][threadIdx.x] + part[1][threadIdx.x] + part[2][threadIdx.x] + part[3][threadIdx.x];
        if (x) atomicAdd(&dst[threadIdx.x], x);
    }
}

// Staging slots of the two-pass permutations for the sorted order perm (sorted slot ->
// user index, device): gpos1 (user index -> staging slot) and gpos2 (sorted slot -> staging
// slot of its user index).  Buckets of 2^shift sorted slots, ordered by user index
// inside a bucket.
int stage_shift_of(int64_t n);
bool build_staging(const int *perm, int64_t n, hipStream_t s, Status &st, int shift, int *gpos1, int *gpos2);

// Root cell when none is given: {x0, y0, side} = (min x, min y, max(range x, range y) (1 + 2^-20)),
// side 1 for a single point; nonfinite when any coordinate is not finite.  Synchronises s.
bool bounding_square(const double2 *xy, int64_t n, hipStream_t s, Status &st, double box[3], bool &nonfinite);

}  // namespace fmm
