// Device to pageable host memory, for arrays that a caller allocates as it
// likes.  A plain copy into such memory runs at 1.5 GB/s into untouched 4 KB
// pages up to 2 MB, 4 GB/s beyond, and 10 GB/s into huge pages, because one
// thread stages the data and takes the destination's page faults one by one as
// it goes.  Here the GPU fills pinned slots, and while it does the caller has
// the system make the destination's pages, a slot at a time, and copies the
// slot before out.  From THREADED bytes on four threads copy and take the
// faults in parallel.  us, plain copy against this one, 4 KB pages: 200 KB 119
// against 25, 1 MB 719 against 88, 2 MB 1302 against 180; huge pages: 4 MB 435
// against 209, 11 MB 1516 against 653, 34 MB 3380 against 1262, 168 MB 16980
// against 5664.  The line: at 11 MB four threads take 660 to 713 us, at 34 MB
// one takes 2493.  Eight threads gain nothing more, and 512 KB slots would limit
// four to 20 GB/s.
#pragma once

#include <hip/hip_runtime.h>
#include <sys/mman.h>
#include <unistd.h>

#include <algorithm>
#include <condition_variable>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <thread>
#include <vector>

#include "pinned.h"

namespace lbmdev {

class HostCopy {
 public:
  HostCopy() = default;
  HostCopy(const HostCopy&) = delete;
  HostCopy& operator=(const HostCopy&) = delete;
  ~HostCopy() {
    for (int i = 0; i < nev_; ++i) (void)hipEventDestroy(ev_[i]);
  }

  // Copies bytes bytes from device memory, after the work queued on st, and
  // returns when they are in dst.  One call at a time.
  hipError_t to_host(void* dst, const void* src, size_t bytes, hipStream_t st) {
    std::lock_guard<std::mutex> one(call_);
    const bool threaded = bytes >= THREADED;
    const size_t slot = threaded ? size_t(1) << 20 : size_t(512) << 10;
    const int nslots = threaded ? MAX_SLOTS : 2;
    const bool once = bytes < SMALL && !called_;
    called_ = true;
    Pinned block;
    char* const pinned = known_to_hip(dst) ? nullptr : (char*)block.take(slot * nslots, !once);
    if (!pinned || !events(nslots, st)) {
      hipError_t e = hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, st);
      const hipError_t w = hipStreamSynchronize(st);
      return e == hipSuccess ? w : e;
    }
    Job j{(char*)dst, (const char*)src, pinned, bytes, slot, nslots, (long)((bytes + slot - 1) / slot), st};
    block.in_use();
    const hipError_t e = threaded ? run_threaded(j) : run(j);
    // an error can leave copies into the slots on the stream
    if (e == hipSuccess || hipStreamSynchronize(st) == hipSuccess) block.done();
    return e;
  }

 private:
  static constexpr size_t THREADED = size_t(16) << 20;
  // New slots cost 84 to 97 us, so an object's first copy makes none, if the
  // library keeps none, for what a plain copy does in 120 us (200 KB; 306 us at
  // 512 KB).
  static constexpr size_t SMALL = size_t(256) << 10;
  static constexpr int THREADS = 4, MAX_SLOTS = 2 * THREADS;

  struct Job {
    char* dst;
    const char* src;
    char* pinned;
    size_t bytes, slot;
    int nslots;
    long chunks;
    hipStream_t st;
  };

  // Memory that HIP allocated or mapped needs no staging.
  static bool known_to_hip(const void* p) {
    hipPointerAttribute_t at;
    if (hipPointerGetAttributes(&at, p) == hipSuccess) return at.type != hipMemoryTypeUnregistered;
    (void)hipGetLastError();
    return false;
  }

  // As many events on st's device, whichever is current.
  bool events(int count, hipStream_t st) {
    if (nev_ >= count) return true;
    int was = 0;
    hipDevice_t own = 0;
    if (hipGetDevice(&was) != hipSuccess || hipStreamGetDevice(st, &own) != hipSuccess) return give_up();
    if (own != was && hipSetDevice(own) != hipSuccess) return give_up();
    hipError_t e = hipSuccess;
    while (nev_ < count && e == hipSuccess) {
      e = hipEventCreateWithFlags(&ev_[nev_], hipEventDisableTiming);
      if (e == hipSuccess) ++nev_;
    }
    if (own != was) (void)hipSetDevice(was);
    return e == hipSuccess || give_up();
  }
  static bool give_up() {
    (void)hipGetLastError();
    return false;
  }

  size_t length(const Job& j, long c) const { return std::min(j.slot, j.bytes - (size_t)c * j.slot); }

  // Only the calling thread queues work: st may name a per-thread stream.
  hipError_t issue(const Job& j, long c) {
    const int k = (int)(c % j.nslots);
    hipError_t e = hipMemcpyAsync(j.pinned + k * j.slot, j.src + (size_t)c * j.slot, length(j, c),
                                  hipMemcpyDeviceToHost, j.st);
    return e == hipSuccess ? hipEventRecord(ev_[k], j.st) : e;
  }

  hipError_t take(const Job& j, long c) {
    const int k = (int)(c % j.nslots);
    const hipError_t e = hipEventSynchronize(ev_[k]);
    if (e == hipSuccess) std::memcpy(j.dst + (size_t)c * j.slot, j.pinned + k * j.slot, length(j, c));
    return e;
  }

  // Makes the pages of chunk c's destination; those that are there, or a system
  // that does not know the request, are no matter.
  void touch(const Job& j, long c) const {
#ifdef MADV_POPULATE_WRITE
    constexpr int request = MADV_POPULATE_WRITE;
#else
    constexpr int request = 23;
#endif
    static const uintptr_t page = (uintptr_t)sysconf(_SC_PAGESIZE);
    char* const to = j.dst + (size_t)c * j.slot;
    const uintptr_t lo = ((uintptr_t)to + page - 1) & ~(page - 1);
    const uintptr_t hi = ((uintptr_t)to + length(j, c)) & ~(page - 1);
    if (lo < hi) (void)madvise((void*)lo, hi - lo, request);
  }

  // All chunks by the calling thread alone.
  hipError_t run(const Job& j) {
    hipError_t e = issue(j, 0);
    for (long c = 0; c < j.chunks && e == hipSuccess; ++c) {
      if (c + 1 < j.chunks) e = issue(j, c + 1);
      if (e != hipSuccess) break;
      touch(j, c);
      e = take(j, c);
    }
    return e;
  }

  // The calling thread keeps the slots filled while the others empty them.
  hipError_t run_threaded(const Job& j) {
    std::mutex m;
    std::condition_variable cv;
    long issued = 0, next = 0;     // chunks queued, chunks taken
    long done[MAX_SLOTS];          // last chunk copied out of each slot
    for (long& d : done) d = -1;
    hipError_t err = hipSuccess;
    auto work = [&]() {
      std::unique_lock<std::mutex> lock(m);
      for (;;) {
        if (next >= j.chunks) return;
        const long c = next++;
        cv.wait(lock, [&]() { return issued > c || err != hipSuccess; });
        if (err != hipSuccess) return;
        lock.unlock();
        const hipError_t e = take(j, c);
        lock.lock();
        if (e != hipSuccess) err = e;
        done[c % j.nslots] = c;
        cv.notify_all();
      }
    };
    // The first chunk waits for all work queued before; the threads start
    // when it has arrived, so none of them spins on a long run.
    hipError_t e = issue(j, 0);
    if (e == hipSuccess) e = hipEventSynchronize(ev_[0]);
    if (e != hipSuccess) return e;
    issued = 1;
    std::vector<std::thread> threads;
    try {
      threads.reserve(THREADS);
      while (threads.size() < THREADS) threads.emplace_back(work);
    } catch (...) {  // no more threads to be had: the ones that run do the work
    }
    if (threads.empty()) return run(j);
    for (long c = 1; c < j.chunks; ++c) {
      std::unique_lock<std::mutex> lock(m);
      cv.wait(lock, [&]() {
        return c < j.nslots || done[c % j.nslots] == c - j.nslots || err != hipSuccess;
      });
      if (err != hipSuccess) break;
      lock.unlock();
      e = issue(j, c);
      lock.lock();
      if (e != hipSuccess) err = e;
      else issued = c + 1;
      cv.notify_all();
      if (err != hipSuccess) break;
    }
    for (std::thread& t : threads) t.join();
    return err;
  }

  std::mutex call_;
  bool called_ = false;
  hipEvent_t ev_[MAX_SLOTS];
  int nev_ = 0;
};

}  // namespace lbmdev
