"""The pool of schedule blocks (pool.hip) on the CPU: its host code against a stand-in for the HIP allocator that counts,
runs out of memory on request, and checks every pointer that it gets back."""
import os
import shutil
import subprocess

import pytest

from paper_1702_02181_amd import build_lib as B

STUB = r'''
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <mutex>
#include <new>
#include <thread>
#include <vector>
#include <hip/hip_runtime_api.h>
#include "pool.h"

static std::mutex mu;
static std::map<void*, size_t> live, pinned;
static size_t device_bytes = 0, limit = ~size_t(0);
static int waits = 0;
static char* next_at = reinterpret_cast<char*>(0x10000000);
static std::atomic<int> refuse{0};  // 1: host allocations fail
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); std::fflush(stdout); std::_Exit(1); } } while (0)

void* operator new(size_t n) { if (refuse) throw std::bad_alloc(); if (void* p = std::malloc(n)) return p; throw std::bad_alloc(); }
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

struct Host {  // the stand-in's own lists may allocate
  std::lock_guard<std::mutex> lk{mu};
  int was = refuse.exchange(0);
  ~Host() { refuse = was; }
};
extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  Host h;
  if (device_bytes + n > limit) return hipErrorOutOfMemory;
  *p = next_at;
  next_at += n + 4096;
  live[*p] = n;
  device_bytes += n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  Host h;
  auto it = live.find(p);
  CHECK(it != live.end());
  waits += it->second == 256;
  device_bytes -= it->second;
  live.erase(it);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { Host h; *p = next_at; next_at += n + 4096; pinned[*p] = n; return hipSuccess; }
hipError_t hipHostFree(void* p) { Host h; CHECK(pinned.erase(p) == 1); return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
}
using namespace fold;
const size_t MB = size_t(1) << 20;

int main(int, char** argv) {
  const std::string what = argv[1];
  if (what == "reuse") {  // a class comes back as the same block; another class does not take it
    void* a = pool_alloc(0, 5 * MB, true);
    pool_free_after_wait(0, a);
    CHECK(waits == 1 && live.size() == 1);
    CHECK(pool_alloc(0, 9 * MB, true) != a);
    CHECK(pool_alloc(1, 5 * MB, true) != a);
    CHECK(pool_alloc(0, 5 * MB, true) == a);
    CHECK(pool_alloc(0, 5 * MB, true) != a);
  } else if (what == "bounds") {  // 1 GiB idle while a schedule is alive, 256 MiB otherwise; the oldest go first
    void* keep = pool_alloc(0, MB, true);
    std::vector<void*> b;
    for (int i = 0; i < 40; ++i) b.push_back(pool_alloc(0, 64 * MB, false));
    for (void* p : b) pool_free(0, p, false);
    CHECK(device_bytes <= kIdleBytes + MB && device_bytes > kIdleBytes - 64 * MB && live.count(b.back()) && !live.count(b[0]));
    pool_free_after_wait(0, keep);
    CHECK(device_bytes <= kIdleBytesUnused);
  } else if (what == "out of memory") {  // idle blocks of other classes go back before an allocation fails
    limit = 100 * MB;
    void* a = pool_alloc(0, 40 * MB, false);
    void* b = pool_alloc(0, 40 * MB, true);
    pool_free(0, a, false);
    CHECK(pool_alloc(0, 56 * MB, false) && live.count(b) && !live.count(a));
    CHECK(!pool_alloc(0, 56 * MB, false));
    pool_free_after_wait(0, b);  // no room for the wait's allocation or room: the block is given back either way
    limit = device_bytes;
    void* c = pool_alloc(0, 40 * MB, true);
    CHECK(c);
    limit = device_bytes;
    pool_free_after_wait(0, c);
    CHECK(!live.count(c));
  } else if (what == "host memory") {  // the lists cannot grow: blocks go back, nothing throws
    std::vector<void*> b;
    for (int i = 0; i < 9; ++i) b.push_back(pool_alloc(0, MB << i, true));
    std::vector<int*> s;
    for (int i = 0; i < 6; ++i) s.push_back(stage_alloc());
    refuse = 1;
    CHECK(!pool_alloc(0, 3 * MB, true));
    for (void* p : b) pool_free(0, p, true);
    for (int* p : s) stage_free(p);
    refuse = 0;
    CHECK(device_bytes <= kIdleBytes && pinned.size() <= kIdleStages);
    CHECK(pool_alloc(0, MB, true));
  } else if (what == "threads") {
    std::vector<std::thread> t;
    for (int k = 0; k < 8; ++k)
      t.emplace_back([k] {
        for (int i = 0; i < 2000; ++i) {
          const size_t n = (size_t)(1 + (i * 7 + k * 13) % 40) * MB;
          void* a = pool_alloc(0, n, true);
          void* b = pool_alloc(0, n / 2, false);
          int* s = stage_alloc();
          CHECK(a && b && a != b && s);
          {
            Host h;
            CHECK(live.at(a) >= n && live.at(b) >= n / 2);
          }
          pool_free(0, b, false);
          stage_free(s);
          pool_free_after_wait(0, a);
        }
      });
    for (auto& x : t) x.join();
    CHECK(device_bytes <= kIdleBytesUnused && pinned.size() <= kIdleStages);
  }TRIM
  std::puts("ok");
  return 0;
}
'''
TRIM = r''' else if (what == "trim") {  // every device's idle blocks and the buffers go back, those handed out stay
    void* a = pool_alloc(0, 8 * MB, true);
    void* b = pool_alloc(1, 16 * MB, false);
    void* c = pool_alloc(0, 32 * MB, false);
    int* s = stage_alloc();
    stage_free(s);
    pool_free(1, b, false);
    pool_free(0, c, false);
    CHECK(pool_trim() == 48 * MB && live.size() == 1 && live.count(a) && pinned.empty());
    CHECK(pool_trim() == 0);
    pool_free_after_wait(0, a);
    CHECK(pool_trim() == 8 * MB && live.empty());
  }'''


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("pool")
    (d / "stub.cpp").write_text(STUB.replace("TRIM", TRIM))
    src = os.path.join(B.CSRC, "pool.hip")
    cxx = shutil.which("g++")
    if cxx is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime_api.h"):
        pytest.skip("no C++ compiler or HIP headers")
    r = subprocess.run([cxx, "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + B.CSRC,
                        str(d / "stub.cpp"), "-x", "c++", src, "-o", str(d / "pool"), "-pthread"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return str(d / "pool")


@pytest.mark.parametrize("what", ["reuse", "bounds", "out of memory", "host memory", "threads", "trim"])
def test_pool(program, what):
    r = subprocess.run([program, what], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", (r.returncode, r.stdout, r.stderr[-500:])
