// Device memory, streams and host pages of plans, kept between plans.
//
// A program that moves its beads makes a plan per step, and hipMalloc and
// hipFree cost by the byte as well as by the call (25 MB: 0.43 ms and 1 ms), a
// pair of streams 0.35 ms.  Blocks of up to POOL_BLOCK bytes are therefore kept
// when they are freed.  With this, one wait per count and tables in one copy, a
// step of 200k beads (6 digits, mixed) went from 10.2 to 3.7 ms: plan 6.5 -> 2.0,
// first matvec 2.0 -> 1.7, free 2.0 -> 0.01.
//   * While a plan is built (a BuildScope on the thread), blocks freed on the way
//     stay with the scope and are handed out again without a wait: everything
//     that touches them is ordered on the scope's one stream.
//   * Otherwise a free requires that the device has finished with the block, as
//     after the wait in rpy_plan_free or at the end of a scope; the block then
//     goes to its device's idle list, for any thread and stream.
//   * Idle blocks of a device are bounded by POOL_IDLE bytes (the longest idle are
//     given back first), those that POOL_AGE plans came and went without are given
//     back, and all of them are when an allocation fails, before it is tried again,
//     or when the program asks for it (rpy_release_memory).
// Larger blocks go straight to hipMalloc and hipFree.  Nothing here throws: where
// the host has no memory for a record, a block is not kept, or not handed out.
#include <algorithm>
#include <map>
#include <mutex>
#include <new>
#include <unordered_map>

#include "pool.h"

namespace rpy {

namespace {
constexpr size_t POOL_BLOCK = (size_t)64 << 20;
constexpr size_t POOL_IDLE = (size_t)256 << 20;
constexpr uint64_t POOL_AGE = 16;
constexpr size_t POOL_LANES = 4;  // idle lanes and idle host pages per device

struct Idle {
  IdleBlock b;
  uint64_t since;  // plans freed before it became idle
};
struct DevPool {
  std::vector<Idle> idle;  // longest idle first
  size_t bytes = 0;
  uint64_t plans = 0;
  std::vector<Lane> lanes;
  std::vector<void*> pages;
};
struct Pool {
  std::mutex mu;
  std::unordered_map<void*, std::pair<size_t, int>> live;  // block -> size, device
  std::map<int, DevPool> dev;
};
// never destroyed: the runtime may be gone by then, and takes the memory with it;
// in storage of its own, so that it is always there
Pool& pool() {
  alignas(Pool) static char at[sizeof(Pool)];
  static Pool* p = new (at) Pool;
  return *p;
}
thread_local BuildScope* t_scope = nullptr;
thread_local bool t_nokeep = false;

int current_device() {
  int d = 0;
  if (hipGetDevice(&d) != hipSuccess) (void)hipGetLastError();
  return d;
}

// sizes in steps of an eighth of their power of two (of 256 bytes at least)
size_t block_size(size_t n) {
  size_t top = 256;
  while (2 * top <= n) top *= 2;
  const size_t step = std::max<size_t>(256, top / 8);
  return (std::max<size_t>(n, 1) + step - 1) / step * step;
}

// the smallest block that holds n and wastes at most half as much again
template <class V, class Get>
void* take_fit(V& v, size_t n, size_t* size, Get block) {
  auto best = v.end();
  for (auto it = v.begin(); it != v.end(); ++it) {
    const size_t s = block(*it).size;
    if (s >= n && s <= n + n / 2 && (best == v.end() || s < block(*best).size)) best = it;
  }
  if (best == v.end()) return nullptr;
  void* p = block(*best).p;
  *size = block(*best).size;
  v.erase(best);
  return p;
}

void give_back(DevPool& d, size_t keep_bytes, uint64_t oldest) {
  size_t k = 0;
  while (k < d.idle.size() && (d.bytes > keep_bytes || d.idle[k].since < oldest)) {
    (void)hipFree(d.idle[k].b.p);
    d.bytes -= d.idle[k].b.size;
    ++k;
  }
  d.idle.erase(d.idle.begin(), d.idle.begin() + k);
}

void make_idle(Pool& P, int dev, const IdleBlock& b) {
  DevPool& d = P.dev[dev];
  d.idle.push_back(Idle{b, d.plans});
  d.bytes += b.size;
  give_back(d, POOL_IDLE, 0);
}
}  // namespace

hipError_t dev_alloc_bytes(void** out, size_t n) {
  *out = nullptr;
  const int dev = current_device();
  size_t size = block_size(n);
  void* p = nullptr;
  try {
    Pool& P = pool();
    if (size <= POOL_BLOCK) {
      if (t_scope && t_scope->device() == dev)
        p = take_fit(t_scope->freed, size, &size, [](const IdleBlock& b) -> const IdleBlock& { return b; });
      if (!p) {
        std::lock_guard<std::mutex> lk(P.mu);
        DevPool& d = P.dev[dev];
        p = take_fit(d.idle, size, &size, [](const Idle& i) -> const IdleBlock& { return i.b; });
        if (p) d.bytes -= size;
      }
    }
    if (!p) {
      hipError_t he = hipMalloc(&p, size);
      if (he == hipErrorOutOfMemory) {
        // give everything idle back, and try once more
        (void)hipGetLastError();
        if (t_scope) t_scope->flush();
        {
          std::lock_guard<std::mutex> lk(P.mu);
          give_back(P.dev[dev], 0, ~(uint64_t)0);
        }
        he = hipMalloc(&p, size);
      }
      if (he != hipSuccess) return he;
    }
    std::lock_guard<std::mutex> lk(P.mu);
    P.live[p] = {size, dev};
  } catch (const std::bad_alloc&) {  // no host memory for the record of the block
    if (p) (void)hipFree(p);
    return hipErrorOutOfMemory;
  }
  *out = p;
  return hipSuccess;
}

// A list that cannot grow does not keep the block.
void dev_free(void* p) {
  if (!p) return;
  Pool& P = pool();
  std::pair<size_t, int> b{0, 0};
  {
    std::lock_guard<std::mutex> lk(P.mu);
    auto it = P.live.find(p);
    if (it != P.live.end()) {
      b = it->second;
      P.live.erase(it);
    }
  }
  // (a block of another device than the current one, which the caller waited for)
  if (b.first > 0 && b.first <= POOL_BLOCK && !t_nokeep && b.second == current_device()) try {
      if (t_scope && t_scope->device() == b.second) {
        t_scope->freed.push_back(IdleBlock{p, b.first});
        return;
      }
      std::lock_guard<std::mutex> lk(P.mu);
      make_idle(P, b.second, IdleBlock{p, b.first});
      return;
    } catch (const std::bad_alloc&) {
    }
  (void)hipFree(p);
}

BuildScope::BuildScope(hipStream_t s) : s_(s), dev_(current_device()), outer_(t_scope) {
  try {
    Pool& P = pool();
    std::lock_guard<std::mutex> lk(P.mu);
    DevPool& d = P.dev[dev_];
    if (!d.pages.empty()) {
      page_ = d.pages.back();
      d.pages.pop_back();
    }
  } catch (const std::bad_alloc&) {
  }
  t_scope = this;
}

BuildScope::~BuildScope() {
  t_scope = outer_;
  const bool done = hipStreamSynchronize(s_) == hipSuccess;
  if (!done) (void)hipGetLastError();
  Pool& P = pool();
  std::lock_guard<std::mutex> lk(P.mu);
  for (const IdleBlock& b : freed) try {
      if (done) make_idle(P, dev_, b);
      else (void)hipFree(b.p);
    } catch (const std::bad_alloc&) {
      (void)hipFree(b.p);
    }
  if (!page_) return;
  try {
    DevPool& d = P.dev[dev_];
    if (done && d.pages.size() < POOL_LANES) {
      d.pages.push_back(page_);
      return;
    }
  } catch (const std::bad_alloc&) {
  }
  (void)hipHostFree(page_);
}

void BuildScope::flush() {
  for (const IdleBlock& b : freed) (void)hipFree(b.p);  // waits for the device
  freed.clear();
}

void* BuildScope::page() {
  if (!page_ && hipHostMalloc(&page_, BUILD_PAGE, hipHostMallocDefault) != hipSuccess) {
    (void)hipGetLastError();
    page_ = nullptr;
  }
  return page_;
}

BuildScope* BuildScope::current() { return t_scope; }

bool device_wait() {
  void* p = nullptr;
  const bool ok = hipMalloc(&p, 256) == hipSuccess && hipFree(p) == hipSuccess;
  if (!ok) (void)hipGetLastError();
  return ok;
}

NoKeep::NoKeep(bool on) : before_(t_nokeep) { t_nokeep = t_nokeep || on; }
NoKeep::~NoKeep() { t_nokeep = before_; }

bool take_lane(int dev, Lane* out) {
  Pool& P = pool();
  std::lock_guard<std::mutex> lk(P.mu);
  const auto it = P.dev.find(dev);
  if (it == P.dev.end() || it->second.lanes.empty()) return false;
  *out = it->second.lanes.back();
  it->second.lanes.pop_back();
  return true;
}

bool keep_lane(int dev, const Lane& l) {
  // a stream that is still part of a capture is not kept
  for (hipStream_t s : {l.near, l.far2}) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) != hipSuccess || st != hipStreamCaptureStatusNone) {
      (void)hipGetLastError();
      return false;
    }
  }
  Pool& P = pool();
  std::lock_guard<std::mutex> lk(P.mu);
  try {
    DevPool& d = P.dev[dev];
    if (d.lanes.size() >= POOL_LANES) return false;
    d.lanes.push_back(l);
  } catch (const std::bad_alloc&) {
    return false;
  }
  return true;
}

void plan_freed(int dev) {
  Pool& P = pool();
  std::lock_guard<std::mutex> lk(P.mu);
  const auto it = P.dev.find(dev);
  if (it == P.dev.end()) return;  // nothing was kept or asked for
  DevPool& d = it->second;
  ++d.plans;
  if (d.plans > POOL_AGE) give_back(d, POOL_IDLE, d.plans - POOL_AGE);
}

void give_idle_back(int dev) {
  Pool& P = pool();
  std::lock_guard<std::mutex> lk(P.mu);
  const auto it = P.dev.find(dev);
  if (it == P.dev.end()) return;
  give_back(it->second, 0, ~(uint64_t)0);
  for (void* q : it->second.pages) (void)hipHostFree(q);
  it->second.pages.clear();
}

}  // namespace rpy
