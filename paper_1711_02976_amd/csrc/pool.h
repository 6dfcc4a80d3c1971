// Device memory, streams and host pages of plans, kept between plans (pool.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <vector>

namespace rpy {

struct IdleBlock {
  void* p;
  size_t size;
};

// Device memory of a plan or of its building.  dev_free outside a BuildScope
// requires that the device has finished with the block.
hipError_t dev_alloc_bytes(void** out, size_t n);
template <class T>
hipError_t dev_alloc(T** out, size_t n) {
  void* p = nullptr;
  const hipError_t e = dev_alloc_bytes(&p, n);
  *out = static_cast<T*>(p);
  return e;
}
void dev_free(void* p);

constexpr size_t BUILD_PAGE = 16384;

// While one lives on a thread, blocks that the thread frees are reused by its
// next allocations without a wait: every use of a block allocated meanwhile must
// be on the scope's stream.  Its end waits for the stream.
class BuildScope {
 public:
  explicit BuildScope(hipStream_t s);
  ~BuildScope();
  BuildScope(const BuildScope&) = delete;
  BuildScope& operator=(const BuildScope&) = delete;
  int device() const { return dev_; }
  void flush();
  void* page();  // BUILD_PAGE bytes of host memory that kernels can write; null if there is none
  static BuildScope* current();
  std::vector<IdleBlock> freed;

 private:
  hipStream_t s_;
  int dev_;
  BuildScope* outer_;
  void* page_ = nullptr;
};

// Waits until the device has finished with everything issued so far, in the one
// way that a capture in relaxed mode on another stream survives (hipFree's own
// wait; hipDeviceSynchronize ends it).  false: refused.
bool device_wait();

// While one lives on a thread, its dev_free calls go to hipFree, which waits for
// the device by itself.
class NoKeep {
 public:
  explicit NoKeep(bool on);
  ~NoKeep();
  NoKeep(const NoKeep&) = delete;
  NoKeep& operator=(const NoKeep&) = delete;

 private:
  bool before_;
};

// The streams and events a plan overlaps its phases with (default priority).
struct Lane {
  hipStream_t near, far2;
  hipEvent_t fork, join, p2m, m2l0;
};
bool take_lane(int dev, Lane* out);         // false: none idle
bool keep_lane(int dev, const Lane& lane);  // idle streams and events; false: not kept
void plan_freed(int dev);                   // a plan's memory has been freed
void give_idle_back(int dev);               // the device's idle blocks and host pages

}  // namespace rpy
