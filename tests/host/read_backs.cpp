// Host check of the page-locked read-back buffers (wino_readback.hpp) with the allocating call replaced: buffers are
// not shared, not handed out again unless given back, at most kReadBacks.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <thread>
#include <vector>

#include "wino_readback.hpp"

static std::atomic<int> allocations{0};
static std::atomic<bool> refuse{false};

extern "C" hipError_t hipHostMalloc(void** p, size_t bytes, unsigned int) {
  if (refuse) return hipErrorOutOfMemory;
  ++allocations;
  *p = std::malloc(bytes);
  return hipSuccess;
}
extern "C" hipError_t hipGetLastError() { return hipSuccess; }

#define CHECK(c) \
  if (!(c)) return std::printf("line %d: %s\n", __LINE__, #c), 1

int main() {
  using wino::ReadBack;
  refuse = true;
  for (int i = 0; i < 100; ++i) {
    ReadBack none;
    CHECK(!none.ptr);
    none.done();
  }
  refuse = false;
  for (int i = 0; i < 1000; ++i) {                   // one at a time: one buffer
    ReadBack b;
    CHECK(b.ptr);
    b.done();
  }
  CHECK(allocations == 1);
  // eight threads use buffers at once, each its own
  std::atomic<bool> shared{false};
  std::vector<std::thread> threads;
  for (int t = 0; t < 12; ++t)
    threads.emplace_back([&, t] {
      for (int i = 0; i < 20000; ++i) {
        ReadBack b;
        if (!b.ptr) continue;
        std::memset(b.ptr, t + 1, ReadBack::kBytes);
        for (size_t j = 0; j < ReadBack::kBytes; j += 64)
          if (static_cast<char*>(b.ptr)[j] != t + 1) shared = true;
        b.done();
      }
    });
  for (auto& t : threads) t.join();
  CHECK(!shared && allocations >= 1 && allocations <= ReadBack::kReadBacks);
  void* lost[ReadBack::kReadBacks];                  // not given back: never seen again
  for (auto& p : lost) {
    ReadBack b;
    CHECK(b.ptr);
    p = b.ptr;
  }
  for (int i = 0; i < ReadBack::kReadBacks; ++i)
    for (int j = 0; j < i; ++j) CHECK(lost[i] != lost[j]);
  ReadBack ninth;
  CHECK(!ninth.ptr && allocations == ReadBack::kReadBacks);
  std::printf("ok\n");
  return 0;
}
