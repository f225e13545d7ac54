// Device memory of the tables, and the memory of closed ones kept for the next.
#pragma once

#include <stddef.h>

#include <mutex>

namespace mlkv {

// A program that opens and closes tables otherwise pays the driver for mapping
// (and clearing) their memory each time, 0.3 to 8 ms for 200 MB, varying within
// a process. At most kPoolBytes are kept, in at most kPoolBlocks blocks: the
// oldest go first, trim() frees all of them, and all of them go before any
// allocation is reported as failed. A block comes back only once nothing on
// the device uses it, and is taken under the lock, so any thread and stream may
// have it. A block remembers the runtime's id of its allocation: one that the
// program freed behind the pool's back (a device reset) is forgotten, neither
// given out nor freed.
constexpr size_t kPoolBytes = 256ull << 20;
constexpr int kPoolBlocks = 64;

class DevicePool {
 public:
  // New device memory, kept blocks freed for it if it does not fit beside them.
  hipError_t alloc(void** p, size_t bytes) {
    *p = nullptr;
    if (bytes == 0) bytes = 256;
    hipError_t e = hipMalloc(p, bytes);
    if (e == hipErrorOutOfMemory && trim() > 0) {
      (void)hipGetLastError();
      e = hipMalloc(p, bytes);
    }
    return e;
  }

  // Memory for `*bytes` on the current device: a kept block at most a quarter
  // larger (*bytes becomes its size), else new memory.
  hipError_t take(void** p, size_t* bytes) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    {
      std::lock_guard<std::mutex> lock(mu_);
      forget_dead();
      int best = -1;
      for (int k = 0; k < n_; ++k)
        if (b_[k].device == dev && b_[k].bytes >= *bytes && b_[k].bytes <= *bytes + *bytes / 4 &&
            (best < 0 || b_[k].bytes < b_[best].bytes))
          best = k;
      if (best >= 0) {
        *p = b_[best].ptr;
        *bytes = b_[best].bytes;
        drop(best);
        return hipSuccess;
      }
    }
    return alloc(p, *bytes);
  }

  // Gives back a block of take() that no queued work uses any more.
  void give(int device, void* p, size_t bytes) {
    if (p == nullptr) return;
    const unsigned long long id = bytes <= kPoolBytes ? id_of(p) : 0;
    if (id == 0) {
      (void)hipFree(p);
      return;
    }
    std::lock_guard<std::mutex> lock(mu_);
    forget_dead();
    free_oldest(kPoolBytes - bytes, kPoolBlocks - 1);
    b_[n_++] = {device, p, bytes, id};
    bytes_ += bytes;
  }

  // Frees every kept block; returns their bytes.
  size_t trim() {
    std::lock_guard<std::mutex> lock(mu_);
    forget_dead();
    const size_t had = bytes_;
    free_oldest(0, 0);
    return had;
  }

 private:
  struct Block {
    int device;
    void* ptr;
    size_t bytes;
    unsigned long long id;
  };

  // The runtime's id of the allocation at p, 0 if there is none.
  static unsigned long long id_of(void* p) {
    unsigned long long id = 0;
    if (hipPointerGetAttribute(&id, HIP_POINTER_ATTRIBUTE_BUFFER_ID, (hipDeviceptr_t)p) == hipSuccess) return id;
    (void)hipGetLastError();
    return 0;
  }
  void drop(int k) {
    bytes_ -= b_[k].bytes;
    for (--n_; k < n_; ++k) b_[k] = b_[k + 1];
  }
  void forget_dead() {
    for (int k = n_ - 1; k >= 0; --k)
      if (id_of(b_[k].ptr) != b_[k].id) drop(k);
  }
  void free_oldest(size_t keep, int blocks) {
    while (bytes_ > keep || n_ > blocks) {
      (void)hipFree(b_[0].ptr);
      drop(0);
    }
  }

  std::mutex mu_;
  Block b_[kPoolBlocks];  // oldest first
  int n_ = 0;
  size_t bytes_ = 0;
};

}  // namespace mlkv
