// Blocks and read-back buffers of the schedules (see pool.h).

#include "pool.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <vector>

namespace fold {

namespace {

struct Idle {
  void* ptr;
  size_t bytes;
};

struct DevicePool {
  std::vector<Idle> idle;  // oldest first
  size_t idle_bytes = 0;
  int alive = 0;
};

struct Pools {
  std::mutex mu;
  std::map<int, DevicePool> device;
  std::map<void*, size_t> handed_out;
  std::vector<int*> stages;
  Pools() { stages.reserve(kIdleStages); }
};

// never destroyed: no HIP call is made after the runtime's own shutdown
Pools& pools() {
  static Pools* p = new Pools;
  return *p;
}

size_t size_class(size_t bytes) {
  size_t step = 1 << 14;  // classes of 64 KB and more: 4, 5, 6, 7 steps
  while (7 * step < bytes) step *= 2;
  return std::max<size_t>(4, (bytes + step - 1) / step) * step;
}

// takes the oldest idle blocks past `keep` bytes out of the pool
std::vector<Idle> trim(DevicePool& d, size_t keep) {
  size_t n = 0, left = d.idle_bytes;
  while (left > keep) left -= d.idle[n++].bytes;
  std::vector<Idle> out(d.idle.begin(), d.idle.begin() + n);
  d.idle.erase(d.idle.begin(), d.idle.begin() + n);
  d.idle_bytes = left;
  return out;
}

size_t release(const std::vector<Idle>& blocks) {
  size_t bytes = 0;
  for (const Idle& b : blocks) {
    bytes += b.bytes;
    (void)hipFree(b.ptr);
  }
  return bytes;
}

// a block of a class that is idle, or NULL
void* take(int device, size_t size, bool lasting) {
  Pools& P = pools();
  std::lock_guard<std::mutex> lk(P.mu);
  DevicePool& d = P.device[device];
  for (size_t i = d.idle.size(); i-- > 0;) {  // the last one given back first
    if (d.idle[i].bytes != size) continue;
    void* p = d.idle[i].ptr;
    P.handed_out[p] = size;
    d.idle_bytes -= size;
    d.idle.erase(d.idle.begin() + i);
    d.alive += lasting;
    return p;
  }
  return nullptr;
}

void* device_alloc(size_t size) {
  void* p = nullptr;
  if (hipMalloc(&p, size) == hipSuccess) return p;
  (void)hipGetLastError();
  return nullptr;
}

}  // namespace

void* pool_alloc(int device, size_t bytes, bool lasting) noexcept {
  const size_t size = size_class(bytes);
  void* p = nullptr;
  try {
    Pools& P = pools();
    if ((p = take(device, size, lasting))) return p;
    p = device_alloc(size);
    if (!p) {
      std::vector<Idle> drop;
      {
        std::lock_guard<std::mutex> lk(P.mu);
        drop = trim(P.device[device], 0);
      }
      release(drop);
      p = device_alloc(size);
    }
    if (!p) return nullptr;
    std::lock_guard<std::mutex> lk(P.mu);
    P.handed_out[p] = size;
    P.device[device].alive += lasting;
    return p;
  } catch (...) {  // no host memory for the pool's own lists
    if (p) (void)hipFree(p);
    return nullptr;
  }
}

void pool_free(int device, void* ptr, bool lasting) noexcept {
  if (!ptr) return;
  Pools& P = pools();
  std::vector<Idle> drop;
  bool kept = false;
  try {
    std::lock_guard<std::mutex> lk(P.mu);
    DevicePool& d = P.device[device];
    auto it = P.handed_out.find(ptr);
    if (it == P.handed_out.end()) return;
    const size_t size = it->second;
    P.handed_out.erase(it);
    d.alive -= lasting;
    d.idle.push_back({ptr, size});
    d.idle_bytes += size;
    kept = true;
    drop = trim(d, d.alive > 0 ? kIdleBytes : kIdleBytesUnused);
  } catch (...) {
    if (!kept) (void)hipFree(ptr);
  }
  release(drop);
}

size_t pool_trim() noexcept {
  std::vector<std::vector<Idle>> drop;
  int* stages[kIdleStages];
  int n = 0;
  try {
    Pools& P = pools();
    std::lock_guard<std::mutex> lk(P.mu);
    drop.reserve(P.device.size());
    for (auto& d : P.device) drop.push_back(trim(d.second, 0));
    for (int* p : P.stages) stages[n++] = p;
    P.stages.clear();
  } catch (...) {  // no host memory for the lists: what was not taken stays idle
  }
  size_t bytes = 0;
  for (const auto& blocks : drop) bytes += release(blocks);
  while (n > 0) (void)hipHostFree(stages[--n]);
  return bytes;
}

// Waits for everything on the current device by freeing a small allocation.  hipDeviceSynchronize would do, but where
// another thread records a stream (a graph of its own, a framework's) it fails and breaks that recording; hipFree, which
// gave the schedules' arrays back before there was a pool, does not.  It costs 13 to 21 us more a schedule (84 ->
// 98 us for a schedule of 152 nodes with its forward; hipMalloc and hipFree of its arrays: 327).
static bool wait_for_device() {
  void* p = nullptr;
  return hipMalloc(&p, 256) == hipSuccess && hipFree(p) == hipSuccess;
}

void pool_free_after_wait(int device, void* ptr) noexcept {
  if (!ptr) return;
  int current = device;
  (void)hipGetDevice(&current);
  if (current != device) (void)hipSetDevice(device);
  const bool waited = wait_for_device();
  if (waited) {
    pool_free(device, ptr, true);
  } else {  // a capture that forbids it, or a device in error: as if there were no pool
    (void)hipGetLastError();
    {
      Pools& P = pools();
      std::lock_guard<std::mutex> lk(P.mu);
      P.handed_out.erase(ptr);
      auto d = P.device.find(device);
      if (d != P.device.end()) d->second.alive -= 1;
    }
    (void)hipFree(ptr);
  }
  if (current != device) (void)hipSetDevice(current);
}

int* stage_alloc() noexcept {
  Pools& P = pools();
  {
    std::lock_guard<std::mutex> lk(P.mu);
    if (!P.stages.empty()) {
      int* p = P.stages.back();
      P.stages.pop_back();
      return p;
    }
  }
  void* p = nullptr;
  if (hipHostMalloc(&p, kStageInts * sizeof(int), hipHostMallocPortable) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  return static_cast<int*>(p);
}

void stage_free(int* p) noexcept {
  if (!p) return;
  Pools& P = pools();
  {
    std::lock_guard<std::mutex> lk(P.mu);
    if (P.stages.size() < P.stages.capacity() && P.stages.size() < (size_t)kIdleStages) {
      P.stages.push_back(p);
      return;
    }
  }
  (void)hipHostFree(p);
}

}  // namespace fold
