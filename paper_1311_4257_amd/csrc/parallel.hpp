// fn(0) .. fn(n - 1) on up to 16 host threads, the caller's among them.  Plain host
// code (no HIP types).
#pragma once

#include <algorithm>
#include <atomic>
#include <cstdint>
#include <exception>
#include <mutex>
#include <thread>
#include <vector>

namespace dfmm {

// An exception of fn ends the loop and comes back to the caller: thrown past a
// thread's start it would end the process.  Threads that cannot be started are
// done without.
template <class F>
void parallel_for(int64_t n, F&& fn) {
  const unsigned hc = std::thread::hardware_concurrency();
  const int64_t nt = std::min<int64_t>(std::min<int64_t>(hc ? hc : 1, 16), n);
  std::atomic<int64_t> next{0};
  std::exception_ptr err;
  std::mutex mu;
  auto work = [&]() {
    try {
      for (int64_t i = next++; i < n; i = next++) fn(i);
    } catch (...) {
      std::lock_guard<std::mutex> lock(mu);
      if (!err) err = std::current_exception();
      next = n;
    }
  };
  std::vector<std::thread> th;
  th.reserve(size_t(std::max<int64_t>(nt, 1)));
  for (int64_t t = 1; t < nt; ++t) try {
      th.emplace_back(work);
    } catch (...) {
      break;
    }
  work();
  for (auto& x : th) x.join();
  if (err) std::rethrow_exception(err);
}

}  // namespace dfmm
