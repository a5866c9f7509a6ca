// Host threads of the coordinate ascent's neuron step and of the exact per-layer optimum.
#pragma once

#include <algorithm>
#include <cstdint>
#include <exception>
#include <mutex>
#include <thread>
#include <vector>

namespace dtp {

// Threads for the neuron steps of `tasks` layers of about `ns` nanoseconds each: one per 200 us of work, about what
// starting and joining one costs several times over, and no more than the host runs at once.
inline int threads_for(int tasks, int64_t ns) {
  const int64_t hw = std::max(1u, std::thread::hardware_concurrency());
  return (int)std::max<int64_t>(1, std::min<int64_t>({tasks * ns / 200000, tasks, hw}));
}

// Runs `work` on n threads, this one among them.  A thread that cannot be started, for want of
// one or of memory, is done without (the others take its share); what any of them throws is
// thrown here, once all have ended.
template <typename F>
void run_on_threads(int n, F&& work) {
  std::mutex mu;
  std::exception_ptr failed;
  auto guarded_work = [&]() {
    try {
      work();
    } catch (...) {
      std::lock_guard<std::mutex> lock(mu);
      failed = std::current_exception();
    }
  };
  std::vector<std::thread> pool;
  try {
    pool.reserve((size_t)n);
    for (int t = 1; t < n; ++t) pool.emplace_back(guarded_work);
  } catch (...) {  // a started thread has to be joined, whatever the reason
  }
  guarded_work();
  for (auto& th : pool) th.join();
  if (failed) std::rethrow_exception(failed);
}

}  // namespace dtp
