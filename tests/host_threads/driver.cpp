// The threads of the neuron step where they cannot all be had: an allocation that fails while
// they are started, and work that throws.  Every task is done once, no thread is left behind
// and the process goes on.
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <new>
#include <stdexcept>
#include <vector>

#include "host_threads.h"

static std::atomic<long> g_allocs_left{-1};  // -1: no limit

static void* take(std::size_t n) {
  if (g_allocs_left >= 0 && g_allocs_left-- <= 0) {
    g_allocs_left = 0;
    throw std::bad_alloc();
  }
  if (void* p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void* operator new(std::size_t n) { return take(n); }
void* operator new[](std::size_t n) { return take(n); }
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }
void operator delete[](void* p) noexcept { std::free(p); }
void operator delete[](void* p, std::size_t) noexcept { std::free(p); }

#define CHECK(cond)                                                             \
  do {                                                                          \
    if (!(cond)) {                                                              \
      std::fprintf(stderr, "FAILED %s:%d: %s\n", __FILE__, __LINE__, #cond);    \
      std::exit(1);                                                             \
    }                                                                           \
  } while (0)

int main() {
  constexpr int kTasks = 64;
  for (long allocs = 0; allocs < 12; ++allocs) {  // from the first allocation to past the last thread's
    std::vector<std::atomic<int>> done(kTasks);
    std::atomic<int> next{0};
    g_allocs_left = allocs;
    dtp::run_on_threads(6, [&]() {
      for (int i = next++; i < kTasks; i = next++) ++done[i];
    });
    g_allocs_left = -1;
    for (auto& d : done) CHECK(d == 1);
  }
  for (int thrower = 0; thrower < 8; ++thrower) {
    std::atomic<int> next{0}, ended{0};
    bool caught = false;
    try {
      dtp::run_on_threads(4, [&]() {
        for (int i = next++; i < 8; i = next++) {
          ++ended;
          if (i == thrower) throw std::runtime_error("task");
        }
      });
    } catch (const std::runtime_error&) {
      caught = true;
    }
    CHECK(caught && ended == 8);
  }
  CHECK(dtp::threads_for(1, 1000000) == 1);
  CHECK(dtp::threads_for(100, 1) == 1);
  const int hw = (int)std::max(1u, std::thread::hardware_concurrency());
  CHECK(dtp::threads_for(1 << 20, 200000) == hw);
  CHECK(dtp::threads_for(2, 1000000) == std::min(2, hw));
  std::printf("thread checks passed\n");
  return 0;
}
