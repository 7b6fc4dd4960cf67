// Page-locked buffers for small read-backs, kept by the process.
#pragma once
#include <hip/hip_runtime_api.h>

#include <atomic>
#include <cstddef>

namespace wino {

// One buffer for one read-back: the copy then goes straight to it (a flex training step of 128 images 16x16, C = K = 128:
// 256 -> 234 us; copy and wait alone 365 -> 358).  At most kReadBacks exist, 8 KB in all: they are handed out to
// the calls under way on all threads, come back when those are done and are kept for the next ones until the
// process ends.  Without a free one, or if none can be had, `ptr` is null and the caller reads back to pageable memory.
class ReadBack {
 public:
  static constexpr size_t kBytes = 1024;
  static constexpr int kReadBacks = 8;
  ReadBack() {
    for (auto& slot : free_)
      if ((ptr = slot.exchange(nullptr))) return;
    if (made_.fetch_add(1) < kReadBacks && allocate()) return;
    made_.fetch_sub(1);
  }
  // Gives the buffer back; only after the copy into it is known to have ended.  A buffer never given back (the
  // wait for the copy failed) is not handed out again: the copy may still arrive.
  void done() {
    if (!ptr) return;
    for (auto& slot : free_) {
      void* none = nullptr;
      if (slot.compare_exchange_strong(none, ptr)) break;          // as many slots as buffers
    }
    ptr = nullptr;
  }
  ReadBack(const ReadBack&) = delete;
  ReadBack& operator=(const ReadBack&) = delete;
  void* ptr = nullptr;

 private:
  bool allocate() {
    if (hipHostMalloc(&ptr, kBytes, hipHostMallocPortable) == hipSuccess) return true;
    ptr = nullptr, (void)hipGetLastError();
    return false;
  }
  static inline std::atomic<void*> free_[kReadBacks]{};
  static inline std::atomic<int> made_{0};
};

}  // namespace wino
