// Device memory and side streams kept between the library's objects.
//
// Trees and workspaces are made and released in loops (time stepping makes and destroys a
// tree per call of rk2.transport and rebuilds it per evaluation), and mapping and unmapping
// device memory costs more than building the tree: for 10^6 particles a tree's life from
// build to destroy took 9.3 ms, of which 5.3 ms were the runtime's allocations and releases
// (its stream-ordered pool returns freed blocks to the device whenever more is free than in
// use, whatever the release threshold says, at 0.1-2 ms a block), and 0.4 ms a stream.
//
//  - A block enters the cache idle: no queued work uses it (its owner has synchronised), so
//    any stream and any thread may take it.
//  - Idle blocks of a device are bounded by kIdleBytes; beyond it the oldest go back to the
//    device at once, and all of them do when an allocation of the library's fails.
//  - The uniform trees' own arrays come from the device's stream-ordered pool, whose release
//    threshold is lifted so that they are not unmapped at every synchronisation.  What lies idle
//    there counts towards the same bound (bound_idle).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>

namespace fmm {

constexpr size_t kIdleBytes = size_t(1) << 30;  // per device (of 288 GiB)
constexpr size_t kIdleStreams = 8;              // per device

// hipMalloc, and hipMallocAsync on stream s, on the current device; where memory is short, again
// after everything held idle has gone back.  (NULL on failure, the runtime's error cleared.)
hipError_t device_malloc(void **p, size_t bytes);
hipError_t pool_malloc(void **p, size_t bytes, hipStream_t s);

// A block of at least `bytes` on the current device: an idle one (at most half of it
// unused), else new memory.
hipError_t block_alloc(void **p, size_t bytes);
// Gives a block back; the device work that used it has completed.  NULL is a no-op.
void block_free(void *p);

// Keeps blocks that the device's default memory pool has taken back (once per device).
void retain_pool(int device);
// Returns to the device what the pool holds idle beyond kIdleBytes less the idle blocks.  Called
// where trees have been built or destroyed, the work that used their arrays completed.
void bound_idle(int device);

// A tree's side stream (default priority, non-blocking) and its fork and join events.
struct SideStream {
    hipStream_t stream = nullptr;
    hipEvent_t fork = nullptr, join = nullptr;
};
hipError_t side_stream_take(int device, SideStream &s);
// Idle (its work has completed).
void side_stream_give(int device, SideStream &s);

}  // namespace fmm
