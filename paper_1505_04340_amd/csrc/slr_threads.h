// Host loops on several threads.
#ifndef SLR_THREADS_H
#define SLR_THREADS_H

#include <algorithm>
#include <atomic>
#include <new>
#include <system_error>
#include <thread>
#include <vector>

namespace slr {

// f(i) for i in [0, n) on the calling thread and up to `threads` - 1 others.  A
// thread that cannot be started is done without.  Returns false when a call
// threw (no later index is begun): an exception that left a thread would end the
// process.
template <class F>
bool run_parallel(int n, int threads, F f) {
  std::atomic<int> next{0};
  std::atomic<bool> ok{true};
  auto worker = [&]() noexcept {
    try {
      for (int i = next++; i < n && ok; i = next++) f(i);
    } catch (...) {
      ok = false;
    }
  };
  std::vector<std::thread> pool;
  try {
    for (int t = 1; t < std::min(threads, n); ++t) pool.emplace_back(worker);
  } catch (const std::system_error &) {
  } catch (const std::bad_alloc &) {
  }
  worker();
  for (std::thread &t : pool) t.join();
  return ok;
}

}  // namespace slr

#endif
