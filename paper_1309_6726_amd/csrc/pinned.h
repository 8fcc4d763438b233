// Pinned host memory, lent for the length of one call.
//
// Allocating a block costs 85 us (1 MB) to 700 us (8 MB), and giving one back to
// HIP waits until the whole device is idle and makes any stream capture in
// progress invalid: where handles owned their blocks, destroying one took 70 ms
// beside a busy stream (6 us without a block) and spoilt a capture.  Every call
// that uses a block ends with its stream synchronised, so the library keeps the
// blocks and a call takes one and puts it back.  At most KEEP of each size stay
// (24 MB in all, until the process ends); what more calls at once had needed goes
// back to HIP.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <mutex>

namespace lbmdev {

class Pinned {
 public:
  Pinned() = default;
  Pinned(const Pinned&) = delete;
  Pinned& operator=(const Pinned&) = delete;
  ~Pinned() { release(); }

  // A block of at least `bytes` (at most 8 MB), kept by the library or, with
  // `allocate`, new; null if there is none.
  void* take(size_t bytes, bool allocate) {
    release();
    kind_ = bytes <= SIZE[0] ? 0 : 1;
    {
      std::lock_guard<std::mutex> lock(pool().m);
      Shelf& s = pool().shelf[kind_];
      if (s.n > 0) mem_ = s.block[--s.n];
    }
    if (!mem_ && allocate && bytes <= SIZE[kind_]) {
      const Unrestricted during;
      if (hipHostMalloc(&mem_, SIZE[kind_], hipHostMallocMapped | hipHostMallocPortable) != hipSuccess) {
        (void)hipGetLastError();
        mem_ = nullptr;
      }
    }
    return mem_;
  }

  // Between these two the GPU may use the block: one released in between (a
  // call that failed) goes back to HIP, which waits for the GPU.
  void in_use() { in_use_ = true; }
  void done() { in_use_ = false; }

 private:
  static constexpr size_t SIZE[2] = {size_t(1) << 20, size_t(8) << 20};
  static constexpr int KEEP[2] = {8, 2};

  struct Shelf {
    void* block[8];
    int n;
  };
  struct Pool {
    std::mutex m;
    Shelf shelf[2] = {};
  };
  static Pool& pool() {
    static Pool p;
    return p;
  }

  // Allocations by this thread leave captures alone that are in progress, of
  // its own or of other threads.
  struct Unrestricted {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    Unrestricted() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~Unrestricted() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
  };

  void release() {
    if (!mem_) return;
    if (!in_use_) {
      std::lock_guard<std::mutex> lock(pool().m);
      Shelf& s = pool().shelf[kind_];
      if (s.n < KEEP[kind_]) {
        s.block[s.n++] = mem_;
        mem_ = nullptr;
      }
    }
    if (mem_) {
      const Unrestricted during;
      (void)hipHostFree(mem_);
    }
    mem_ = nullptr;
    in_use_ = false;
  }

  void* mem_ = nullptr;
  int kind_ = 0;
  bool in_use_ = false;
};

}  // namespace lbmdev
