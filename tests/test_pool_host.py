"""The memory kept between plans (csrc/pool.hip, host code only) on the CPU, with
the runtime calls it makes replaced by counting ones: bounds on what stays idle,
age, what is given back when an allocation fails, devices, scopes, threads (under
ThreadSanitizer), and host allocations that fail one after another, none of which
may leave an exception or a lost block behind.
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1711_02976_amd", "csrc")

RUNTIME = r"""
#pragma once
#include <cstddef>
#include <cstdint>
typedef enum { hipSuccess = 0, hipErrorOutOfMemory = 2, hipErrorUnknown = 999 } hipError_t;
typedef void* hipStream_t;
typedef void* hipEvent_t;
typedef enum { hipStreamCaptureStatusNone = 0, hipStreamCaptureStatusActive = 1 } hipStreamCaptureStatus;
enum { hipHostMallocDefault = 0 };
hipError_t hipGetDevice(int*);
hipError_t hipMalloc(void**, size_t);
hipError_t hipFree(void*);
hipError_t hipHostMalloc(void**, size_t, unsigned);
hipError_t hipHostFree(void*);
hipError_t hipGetLastError();
hipError_t hipStreamSynchronize(hipStream_t);
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus*);
"""

DRIVER = r"""
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <set>
#include <string>
#include <thread>
#include <vector>
#include "pool.h"
using namespace rpy;
typedef long long ll;

// the device: addresses that are only numbers, a capacity, and what is in use
struct Dev {
  std::mutex mu;
  std::map<void*, size_t> blocks;
  size_t used = 0, cap = (size_t)1 << 40;
  int mallocs = 0;
  std::atomic<int> pages{0};
  uintptr_t next = 0x1000;
} D;
thread_local int cur = 0, own = 0;  // own: the harness's allocations do not fail
bool sync_ok = true, capturing = false;
std::atomic<ll> left{-1};  // host allocations until the next one fails (-1: none does)
void* operator new(size_t n) {
  if (!own && left >= 0 && left-- == 0) throw std::bad_alloc();
  void* p = std::malloc(n);
  if (!p) std::abort();
  return p;
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }
struct Own {
  Own() { ++own; }
  ~Own() { --own; }
};
hipError_t hipGetDevice(int* d) { return *d = cur, hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) {
  Own o;
  std::lock_guard<std::mutex> lk(D.mu);
  if (D.used + n > D.cap) return hipErrorOutOfMemory;
  *p = (void*)D.next;
  D.next += n;
  D.blocks[*p] = n;
  D.used += n;
  ++D.mallocs;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  Own o;
  std::lock_guard<std::mutex> lk(D.mu);
  if (!D.blocks.count(p)) std::printf("freed twice\n"), std::fflush(stdout), std::abort();
  D.used -= D.blocks[p];
  D.blocks.erase(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return *p = std::malloc(n), ++D.pages, hipSuccess; }
hipError_t hipHostFree(void* p) { return std::free(p), --D.pages, hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return sync_ok ? hipSuccess : hipErrorUnknown; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  return *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone, hipSuccess;
}

#define CHECK(c) ((c) ? (void)0 : (std::printf("line %d: %s\n", __LINE__, #c), std::fflush(stdout), std::_Exit(1)))
const size_t MB = (size_t)1 << 20;
char* get(size_t n) {
  void* p = nullptr;
  CHECK(dev_alloc_bytes(&p, n) == hipSuccess && p);
  return (char*)p;
}

void bounds() {
  dev_free(nullptr);
  // a large block is not kept; of small ones at most 256 MB, the longest idle go first
  dev_free(get(65 * MB));
  CHECK(D.used == 0);
  std::vector<char*> v;
  for (int i = 0; i < 10; ++i) v.push_back(get(48 * MB));
  for (char* p : v) dev_free(p);
  CHECK(D.used == 240 * MB && D.mallocs == 11 && !D.blocks.count(v[4]) && D.blocks.count(v[5]));
  // a kept block is handed out again if no more than a third of it is waste; sizes
  // are in steps of an eighth of their power of two
  char* p = get(31 * MB);
  CHECK(D.mallocs == 11);
  char* q = get(29 * MB);
  CHECK(D.mallocs == 12 && D.blocks[q] == 30 * MB);
  char* r = get(0);
  CHECK(D.blocks[r] == 256);
  dev_free(p);
  dev_free(q);
  dev_free(r);
  CHECK(D.used <= 256 * MB);
  // what 16 plans come and go without is given back; what they use is not
  for (int i = 0; i < 17; ++i) {
    dev_free(get(256));
    plan_freed(0);
  }
  CHECK(D.used == 256);
  for (int i = 0; i < 17; ++i) plan_freed(0);
  CHECK(D.used == 0 && D.blocks.empty());
}

void failure() {
  D.cap = 200 * MB;
  std::vector<char*> v;
  for (int i = 0; i < 4; ++i) v.push_back(get(40 * MB));
  dev_free(v[0]);
  dev_free(v[1]);
  char* big = get(90 * MB);  // needs the idle blocks' room
  CHECK(D.used == 80 * MB + D.blocks[big]);
  {
    BuildScope s(nullptr);  // and the scope's
    dev_free(v[2]);
    dev_free(v[3]);
    CHECK(s.freed.size() == 2);
    char* again = get(90 * MB);
    CHECK(s.freed.empty());
    void* none = (void*)1;
    CHECK(dev_alloc_bytes(&none, 100 * MB) == hipErrorOutOfMemory && none == nullptr);
    dev_free(again);
  }
  dev_free(big);
  CHECK(D.used == 0);
}

void scopes() {
  char *a = get(3 * MB), *b = nullptr;
  void* page = nullptr;
  {
    BuildScope s(nullptr);
    CHECK(BuildScope::current() == &s);
    page = s.page();
    CHECK(page && s.page() == page);
    dev_free(a);
    CHECK(get(3 * MB) == a);  // at once, on the scope's stream
    dev_free(a);
    std::thread([&] { b = get(3 * MB); }).join();  // no other thread sees it before the end
    CHECK(b != a);
    cur = 1;  // another device's turn: neither the scope's nor kept
    char* c = get(3 * MB);
    CHECK(c != a);
    cur = 0;
    dev_free(c);
    CHECK(!D.blocks.count(c) && s.freed.size() == 1);
  }
  CHECK(!BuildScope::current() && get(3 * MB) == a);
  {
    BuildScope s(nullptr);
    CHECK(s.page() == page);
    sync_ok = false;  // the wait fails: nothing of the scope is kept
    dev_free(a);
  }
  sync_ok = true;
  CHECK(!D.blocks.count(a) && D.pages == 0);
  {
    const NoKeep n(true);
    const NoKeep m(false);
    dev_free(b);
  }
  CHECK(D.used == 0);
  // lanes: four are kept, none of a capture
  Lane l{&a, &b, nullptr, nullptr, nullptr, nullptr}, o{};
  CHECK(!take_lane(0, &o));
  capturing = true;
  CHECK(!keep_lane(0, l));
  capturing = false;
  for (int i = 0; i < 4; ++i) CHECK(keep_lane(0, l));
  CHECK(!keep_lane(0, l) && !take_lane(1, &o) && take_lane(0, &o) && o.near == l.near);
}

void threads() {
  std::mutex mu;
  std::set<char*> held;
  std::vector<std::thread> ts;
  for (int t = 0; t < 4; ++t)
    ts.emplace_back([&, t] {
      unsigned x = 12345u + t;
      std::vector<char*> mine;
      for (int it = 0; it < 400; ++it) {
        BuildScope* s = it % 7 == 0 ? new BuildScope(nullptr) : nullptr;
        if (s) (void)s->page();
        for (int k = 0; k < 6; ++k) {
          x = x * 1664525u + 1013904223u;
          if ((x >> 16) % 3 || mine.empty()) {
            char* p = get((x >> 8) % (4 * MB));
            std::lock_guard<std::mutex> lk(mu);
            CHECK(held.insert(p).second);
            mine.push_back(p);
          } else {
            {
              std::lock_guard<std::mutex> lk(mu);
              held.erase(mine.back());
            }
            dev_free(mine.back());
            mine.pop_back();
          }
        }
        delete s;
        plan_freed(0);
      }
      for (char* p : mine) {
        {
          std::lock_guard<std::mutex> lk(mu);
          held.erase(p);
        }
        dev_free(p);
      }
    });
  for (auto& t : ts) t.join();
  CHECK(D.used <= 256 * MB && D.pages <= 4);
}

// What the program asks back: idle blocks and pages of one device, nothing in use.
void release() {
  give_idle_back(0);  // a device that the pool has no record of
  char *a = get(3 * MB), *b = get(5 * MB), *c = nullptr;
  {
    BuildScope s(nullptr);
    CHECK(s.page());
    dev_free(a);
    give_idle_back(0);  // a scope's blocks are in use
    CHECK(s.freed.size() == 1 && D.blocks.count(a) && D.pages == 1);
  }
  cur = 1;
  c = get(2 * MB);
  dev_free(c);
  cur = 0;
  CHECK(D.used == 10 * MB);
  give_idle_back(0);
  CHECK(D.used == 7 * MB && D.blocks.count(b) && D.blocks.count(c) && D.pages == 0);
  dev_free(b);
  CHECK(get(5 * MB) == b);  // kept again
  dev_free(b);
  give_idle_back(1);
  give_idle_back(0);
  CHECK(D.used == 0 && D.blocks.empty());
}

// Every host allocation of a plan's course fails in turn.
void no_host_memory() {
  for (ll k = 0; k < 60; ++k) {
    const size_t before = D.blocks.size();
    std::vector<char*> v;
    size_t lost = 0;
    {
      Own o;
      v.reserve(16);
    }
    left = k;
    {
      BuildScope s(nullptr);
      (void)s.page();
      for (int i = 0; i < 8; ++i) {
        void* p = nullptr;
        if (dev_alloc_bytes(&p, (size_t)(1 + i) << 16) == hipSuccess) v.push_back((char*)p);
        else CHECK(!p);
      }
      while (v.size() > 4) {
        dev_free(v.back());
        v.pop_back();
      }
    }
    Lane l{&lost, &lost, nullptr, nullptr, nullptr, nullptr}, o{};
    if (keep_lane(0, l)) CHECK(take_lane(0, &o) && o.near == &lost);
    cur = (int)k + 2;  // a device that the pool has no record of
    CHECK(!take_lane(cur, &o));
    plan_freed(cur);
    { BuildScope s(nullptr); }
    cur = 0;
    for (char* p : v) dev_free(p);
    left = -1;
    // all of it is idle or given back: 17 plans later nothing is in use
    for (int i = 0; i < 18; ++i) plan_freed(0);
    CHECK(D.blocks.empty() && before == 0);
  }
}

int main(int, char** argv) {
  const std::string t = argv[1];
  t == "bounds" ? bounds() : t == "release" ? release() : t == "failure" ? failure() : t == "scopes" ? scopes() : t == "threads" ? threads() : no_host_memory();
  std::printf("ok\n");
}
"""


def _build(tmp, san):
    os.makedirs(tmp / "hip", exist_ok=True)
    (tmp / "hip" / "hip_runtime.h").write_text(RUNTIME)
    (tmp / "driver.cpp").write_text(DRIVER)
    exe = tmp / ("pool_" + (san or "plain"))
    flags = [f"-fsanitize={san}"] if san else []
    subprocess.run(["g++", "-std=c++17", "-g", "-O1", "-pthread", *flags, f"-I{tmp}", f"-I{CSRC}", "-x", "c++",
                    os.path.join(CSRC, "pool.hip"), str(tmp / "driver.cpp"), "-o", str(exe)], check=True)
    return exe


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    return _build(tmp_path_factory.mktemp("pool"), None)


@pytest.mark.parametrize("what", ["bounds", "release", "failure", "scopes", "threads", "no_host_memory"])
def test_kept_memory(exe, what):
    r = subprocess.run([str(exe), what], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr


def test_kept_memory_threads_sanitized(tmp_path):
    try:
        exe = _build(tmp_path, "thread")
    except subprocess.CalledProcessError:
        pytest.skip("no ThreadSanitizer runtime")
    r = subprocess.run([str(exe), "threads"], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
