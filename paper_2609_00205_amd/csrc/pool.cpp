// Memory of one call kept for the next: device buffers and pinned host
// buffers of calls that wait for their stream before they return (the
// container's writers and readers).  hipMalloc and hipFree of a call's ten
// buffers and its plan took 4 of the 8.8 ms of reading a 512^3 FP32
// container, and nearly all of a small one's 1.3 ms.
//
// A block goes back only when no work on it is pending, so any thread and
// any stream may take it next.  The pool holds at most kPoolDevice bytes on a
// GPU (less than 1% of its memory) and kPoolHost of pinned memory, gives back
// what no call took for kPoolIdle when a later call looks, everything when
// an allocation of the library fails (which is then tried again), and all of
// it on request (bm_release_memory).

#include <chrono>
#include <mutex>
#include <vector>

#include "internal.h"

namespace bm {
namespace {

using clk = std::chrono::steady_clock;

constexpr size_t kPoolDevice = size_t(2) << 30, kPoolHost = size_t(64) << 20;
constexpr std::chrono::seconds kPoolIdle{5};

struct Block {
  void* p;
  size_t bytes;
  int device;   // -1: pinned host memory
  clk::time_point since;
};

struct Pool {
  std::mutex mu;
  std::vector<Block> idle;   // in the order they came back
};

// (never destroyed: a call may still run while the process ends)
Pool& pool() {
  static Pool* p = new Pool;
  return *p;
}

void free_block(void* p, int device) {
  if (device < 0)
    (void)hipHostFree(p);
  else
    (void)hipFree(p);
}

void give_back(const std::vector<Block>& blocks) {
  for (const Block& b : blocks) free_block(b.p, b.device);
}

// Moves the blocks that nothing took for kPoolIdle, and the oldest ones of a
// kind over its bound, from the pool to `out`, which has room for every block
// (a failure half way would leave a block with two owners or none).  The
// caller holds the mutex.
void expire(Pool& P, std::vector<Block>& out) {
  const auto old = clk::now() - kPoolIdle;
  for (size_t i = 0; i < P.idle.size();) {
    size_t held = 0;   // of this block's kind, this one and newer ones
    for (size_t j = i; j < P.idle.size(); ++j)
      if (P.idle[j].device == P.idle[i].device) held += P.idle[j].bytes;
    if (P.idle[i].since < old || held > (P.idle[i].device < 0 ? kPoolHost : kPoolDevice)) {
      out.push_back(P.idle[i]);
      P.idle.erase(P.idle.begin() + long(i));
    } else {
      ++i;
    }
  }
}

void* fresh(size_t bytes, bool host) {
  void* p = nullptr;
  if (!host) {
    dev_malloc_bytes(&p, bytes);
    return p;
  }
  hipError_t e = hipHostMalloc(&p, bytes, hipHostMallocDefault);
  if (e == hipErrorOutOfMemory) {
    (void)hipGetLastError();
    pool_release();
    e = hipHostMalloc(&p, bytes, hipHostMallocDefault);
  }
  check_hip(e, "hipHostMalloc");
  return p;
}

}  // namespace

void dev_malloc_bytes(void** p, size_t bytes) {
  hipError_t e = hipMalloc(p, bytes);
  if (e == hipErrorOutOfMemory) {
    (void)hipGetLastError();
    pool_release();
    e = hipMalloc(p, bytes);
  }
  check_hip(e, "hipMalloc");
}

PoolMem pool_take(size_t bytes, bool host) {
  int device = -1;
  if (!host) BM_HIP(hipGetDevice(&device));
  // rounded up so that the next call's slightly different sizes fit
  const size_t step = bytes < (size_t(1) << 20) ? 4096 : size_t(1) << 20;
  bytes = (bytes + step - 1) / step * step;
  std::vector<Block> out;
  PoolMem m;
  {
    Pool& P = pool();
    std::lock_guard<std::mutex> lock(P.mu);
    out.reserve(P.idle.size());
    size_t best = P.idle.size();
    for (size_t i = 0; i < P.idle.size(); ++i) {
      const Block& b = P.idle[i];
      if (b.device == device && b.bytes >= bytes && b.bytes <= bytes + bytes / 2 &&
          (best == P.idle.size() || b.bytes < P.idle[best].bytes))
        best = i;
    }
    if (best < P.idle.size()) {
      m = {P.idle[best].p, P.idle[best].bytes, device};
      P.idle.erase(P.idle.begin() + long(best));
    }
    expire(P, out);
  }
  give_back(out);
  if (!m.p) m = {fresh(bytes, host), bytes, device};
  return m;
}

void pool_put(const PoolMem& m) noexcept {
  if (!m.p) return;
  std::vector<Block> out;
  bool kept = false;
  try {
    Pool& P = pool();
    std::lock_guard<std::mutex> lock(P.mu);
    out.reserve(P.idle.size() + 1);
    P.idle.push_back({m.p, m.bytes, m.device, clk::now()});
    kept = true;
    expire(P, out);
  } catch (...) {   // (no room for the lists: the block was not taken in)
  }
  if (!kept) free_block(m.p, m.device);
  give_back(out);
}

void pool_release() {
  std::vector<Block> out;
  {
    Pool& P = pool();
    std::lock_guard<std::mutex> lock(P.mu);
    out.swap(P.idle);
  }
  give_back(out);
}

}  // namespace bm
