"""The pool of the container calls (csrc/pool.cpp) on the CPU: the file is
compiled by itself against stand-ins for the runtime's allocators, the clock
and operator new, so that its bounds, its expiry and its behaviour when
memory runs out can be reached.  Every block has one owner at any time:
handed out, idle in the pool, or given back."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_00205_amd", "csrc")

MAIN = r"""
#define __HIP_PLATFORM_AMD__ 1
#include <hip/hip_runtime.h>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <new>
#include <set>
#include <unistd.h>

// what internal.h's device functions name (none is called here)
inline unsigned __umulhi(unsigned a, unsigned b) { return unsigned((unsigned long long)(a) * b >> 32); }
using std::isfinite;
#include "pool.cpp"

static long clock_s = 0;                 // the clock
static long fail_new = -1;               // allocations until operator new fails once
static int fail_hip = 0;                 // device / pinned allocations that fail next
static size_t held[2] = {0, 0};          // bytes allocated: device, pinned
static std::map<void*, std::pair<int, size_t>>* live = nullptr;
static uintptr_t next_ptr = 1 << 20;

std::chrono::steady_clock::time_point std::chrono::steady_clock::now() noexcept {
  return time_point(std::chrono::seconds(clock_s));
}

void* operator new(size_t n) {
  if (fail_new >= 0 && fail_new-- == 0) throw std::bad_alloc();
  return malloc(n ? n : 1);
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }

#define CHECK(c) do { if (!(c)) { printf("line %d: %s\n", __LINE__, #c); fflush(stdout); _exit(1); } } while (0)

static hipError_t get(void** p, size_t n, int kind) {
  if (fail_hip > 0) {
    --fail_hip;
    return hipErrorOutOfMemory;
  }
  const long f = fail_new;
  fail_new = -1;
  *p = reinterpret_cast<void*>(next_ptr);
  next_ptr += 4096;
  (*live)[*p] = {kind, n};
  held[kind] += n;
  fail_new = f;
  return hipSuccess;
}
static hipError_t put(void* p, int kind) {
  auto it = live->find(p);
  CHECK(it != live->end());              // freed once
  CHECK(it->second.first == kind);
  held[kind] -= it->second.second;
  live->erase(it);
  return hipSuccess;
}
extern "C" {
hipError_t hipMalloc(void** p, size_t n) { return get(p, n, 0); }
hipError_t hipFree(void* p) { return put(p, 0); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return get(p, n, 1); }
hipError_t hipHostFree(void* p) { return put(p, 1); }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
}
namespace bm {
void check_hip(hipError_t e, const char*) {
  if (e != hipSuccess) throw Error{BM_EHIP, "hip"};
}
}  // namespace bm

using bm::PoolMem;
static const size_t MB = size_t(1) << 20, GB = size_t(1) << 30;

static void bounds() {
  PoolMem m[6];
  for (auto& b : m) b = bm::pool_take(GB, false);
  CHECK(held[0] == 6 * GB);
  for (auto& b : m) bm::pool_put(b);
  CHECK(held[0] == 2 * GB);              // the newest two
  PoolMem h[8];
  for (auto& b : h) b = bm::pool_take(20 * MB, true);
  for (auto& b : h) bm::pool_put(b);
  CHECK(held[1] == 60 * MB && held[0] == 2 * GB);
  PoolMem big = bm::pool_take(3 * GB, false);
  bm::pool_put(big);                     // more than the bound by itself: not kept
  CHECK(held[0] <= 2 * GB);
  bm::pool_release();
  CHECK(held[0] == 0 && held[1] == 0 && live->empty());
}

static void sizes() {
  PoolMem a = bm::pool_take(10 * MB, false);
  void* const p = a.p;
  bm::pool_put(a);
  PoolMem small = bm::pool_take(6 * MB, false);        // 10 > 1.5 x 6
  CHECK(small.p != p);
  PoolMem fit = bm::pool_take(7 * MB, false);
  CHECK(fit.p == p && fit.bytes == 10 * MB);
  PoolMem pinned = bm::pool_take(7 * MB, true);        // another kind
  CHECK(pinned.p != p);
  bm::pool_put(small);
  bm::pool_put(fit);
  bm::pool_put(pinned);
  CHECK(bm::pool_take(10 * MB, false).p == p);
}

static void expiry() {
  PoolMem a = bm::pool_take(8 * MB, false), b = bm::pool_take(64 * MB, false);
  bm::pool_put(a);
  clock_s += 3;
  bm::pool_put(b);
  clock_s += 3;                          // a idle for 6 s, b for 3
  PoolMem c = bm::pool_take(MB, true);   // any call looks
  CHECK(held[0] == 64 * MB);
  clock_s += 3;
  bm::pool_put(c);
  CHECK(held[0] == 0 && held[1] == MB);
}

static void retry() {
  PoolMem a = bm::pool_take(GB, false);
  bm::pool_put(a);
  fail_hip = 1;                          // fails until the pool has given back
  PoolMem b = bm::pool_take(4 * GB, false);
  CHECK(b.p && held[0] == 4 * GB);
  bm::pool_put(b);
  CHECK(held[0] == 0);
  // what the rest of the library allocates, too; and nothing but a lack of memory is tried again
  PoolMem c = bm::pool_take(GB, false);
  bm::pool_put(c);
  fail_hip = 1;
  double* plan = nullptr;
  bm::dev_malloc(&plan, 8 * GB);
  CHECK(plan && held[0] == 8 * GB);
  fail_hip = 2;
  bool threw = false;
  try {
    bm::pool_take(GB, false);
  } catch (const bm::Error&) {
    threw = true;
  }
  CHECK(threw);
}

// operator new fails at every point of a call in turn
static void no_memory() {
  for (long k = 0; k < 8; ++k)
    for (int put = 0; put < 2; ++put) {
      bm::pool_release();
      PoolMem m[5];
      for (auto& b : m) b = bm::pool_take(GB / 2, false);
      PoolMem x = bm::pool_take(GB / 2 + MB, false);
      for (auto& b : m) bm::pool_put(b);               // four kept: the bound is reached
      clock_s += 2;
      PoolMem got;
      fail_new = k;
      if (put) {
        bm::pool_put(x);                               // moves the oldest out
      } else {
        clock_s += 10;                                 // expires all but what it takes
        try {
          got = bm::pool_take(GB / 2, false);
        } catch (const std::bad_alloc&) {
        }
      }
      fail_new = -1;
      std::set<void*> mine;                            // handed out: none twice, all allocated
      if (got.p) mine.insert(got.p);
      if (!put) mine.insert(x.p);
      for (int i = 0; i < 8; ++i) {
        PoolMem t = bm::pool_take(GB / 2, false);
        CHECK(live->count(t.p) == 1);
        CHECK(mine.insert(t.p).second);
      }
      if (!put) bm::pool_put(x);
      if (got.p) bm::pool_put(got);
      for (void* p : mine)
        if (p != got.p && (put || p != x.p)) bm::pool_put(PoolMem{p, (*live)[p].second, 0});
      bm::pool_release();
      CHECK(live->empty());                            // none lost either
    }
}

int main(int, char** argv) {
  live = new std::map<void*, std::pair<int, size_t>>;
  if (!strcmp(argv[1], "bounds")) bounds();
  if (!strcmp(argv[1], "sizes")) sizes();
  if (!strcmp(argv[1], "expiry")) expiry();
  if (!strcmp(argv[1], "retry")) retry();
  if (!strcmp(argv[1], "no_memory")) no_memory();
  puts("ok");
  fflush(stdout);
  _exit(0);
}
"""


@pytest.fixture(scope="module")
def prog(tmp_path_factory):
    d = tmp_path_factory.mktemp("pool")
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "pool")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    r = subprocess.run([shutil.which("g++") or "c++", "-std=c++17", "-O1", "-w", "-I", os.path.join(rocm, "include"),
                        "-I", os.path.join(ROOT, "include"), "-I", CSRC, str(d / "main.cpp"), "-o", exe, "-pthread"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


@pytest.mark.parametrize("what", ["bounds", "sizes", "expiry", "retry", "no_memory"])
def test_pool(prog, what):
    r = subprocess.run([prog, what], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.endswith("ok\n"), (r.returncode, r.stdout, r.stderr)
