// Device memory kept between block handles (host code only).
#pragma once

#include <hip/hip_runtime_api.h>
#include <stddef.h>

#include <mutex>
#include <vector>

// Device memory of destroyed handles and of the build's scratch, kept for the next build: hipMalloc and hipFree cost more
// than the kernels of a small build.  At most 64 MiB in 16 blocks; what does not fit is freed at once, and everything kept is
// given back when an allocation fails.  A block enters only when no work can still use it, so any stream or thread may
// take it.
class DevicePool {
 public:
  static DevicePool &get() {
    static DevicePool *p = new DevicePool();  // never destroyed: the runtime may be gone when static destructors run
    return *p;
  }
  // bytes is rounded up; *got receives the size to hand back to give()
  void *take(int device, size_t bytes, size_t *got) {
    const size_t unit = bytes < ((size_t)1 << 20) ? (size_t)1 << 16 : (size_t)1 << 20;
    bytes = (bytes + unit - 1) / unit * unit;
    {
      std::lock_guard<std::mutex> l(mu_);
      size_t best = blocks_.size();
      for (size_t i = 0; i < blocks_.size(); ++i)
        if (blocks_[i].device == device && blocks_[i].bytes >= bytes && blocks_[i].bytes <= 4 * bytes &&
            (best == blocks_.size() || blocks_[i].bytes < blocks_[best].bytes))
          best = i;
      if (best < blocks_.size()) {
        void *p = blocks_[best].p;
        *got = blocks_[best].bytes;
        total_ -= *got;
        blocks_.erase(blocks_.begin() + (long)best);
        return p;
      }
    }
    void *p = nullptr;
    if (hipMalloc(&p, bytes) != hipSuccess) {
      // the runtime keeps a failure as the thread's last error, where a later look at the launches would find it: the returned
      // pointer alone says whether there is memory
      (void)hipGetLastError();
      release();
      if (hipMalloc(&p, bytes) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
      }
    }
    *got = bytes;
    return p;
  }
  void give(int device, void *p, size_t bytes) {
    {
      std::lock_guard<std::mutex> l(mu_);
      if (blocks_.size() < 16 && total_ + bytes <= ((size_t)64 << 20)) {
        blocks_.push_back(Block{p, bytes, device});
        total_ += bytes;
        return;
      }
    }
    (void)hipFree(p);
  }
  // Waits for all work on the current device.  By freeing a small allocation: hipFree waits for the device, and in a relaxed or
  // another thread's stream capture it is allowed, where hipDeviceSynchronize invalidates the capture.  (Build, read-out and
  // destruction of 62k tokens: 123 us, as with hipDeviceSynchronize; freeing the arrays themselves 166 us.)
  static bool wait_idle() {
    void *p = nullptr;
    if (hipMalloc(&p, 256) == hipSuccess) return hipFree(p) == hipSuccess;
    (void)hipGetLastError();
    return false;
  }

 private:
  struct Block { void *p; size_t bytes; int device; };
  void release() {
    std::lock_guard<std::mutex> l(mu_);
    for (const Block &b : blocks_) (void)hipFree(b.p);
    blocks_.clear();
    total_ = 0;
  }
  std::mutex mu_;
  std::vector<Block> blocks_;
  size_t total_ = 0;
};
