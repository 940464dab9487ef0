// Memory that schedules come and go with: device blocks and pinned read-back buffers kept for the next schedule.
//
// A schedule lives for a batch.  hipMalloc and hipFree of its arrays cost more than its kernels on a small batch (and
// up to milliseconds for the 0.2 GB of a 2 M-node one), and a copy into pageable memory goes through a staging buffer.
// Blocks are handed out whole by size class (four to a power of two, so at most a quarter is unused), under one lock,
// to any thread; a block comes back only when the GPU has finished with it.  At most kIdleBytes per device stay idle,
// kIdleBytesUnused once no schedule is alive there, and none after pool_trim or when an allocation of the pool's own fails
// for want of memory.  Nothing here throws: what cannot be kept for want of host memory is given back at once.
#pragma once

#include <cstddef>

namespace fold {

constexpr size_t kIdleBytes = size_t(1) << 30, kIdleBytesUnused = size_t(256) << 20;

// A device block of at least `bytes` on the current device (`device`), or NULL.  `lasting`: counted as alive until
// pool_free (a schedule's arrays, in contrast to a call's temporaries).
void* pool_alloc(int device, size_t bytes, bool lasting) noexcept;
// Gives a block back.  The caller has waited for every use of it.
void pool_free(int device, void* ptr, bool lasting) noexcept;
// Waits for the device (as hipFree would), then gives a lasting block back.
void pool_free_after_wait(int device, void* ptr) noexcept;
// Gives every idle block and read-back buffer of all devices back to the system; returns the device bytes.
size_t pool_trim() noexcept;

// A pinned host buffer of kStageInts ints that kernels write, or NULL; at most kIdleStages stay idle.
constexpr size_t kStageInts = 33536;
constexpr int kIdleStages = 4;
int* stage_alloc() noexcept;
void stage_free(int* p) noexcept;

}  // namespace fold
