// parallel_for (csrc/parallel.hpp): every index once, and exceptions of the loop's
// body in the caller.
#include "parallel.hpp"

#include <cstdio>
#include <new>
#include <stdexcept>

#define CHECK(x)                                              \
  do {                                                        \
    if (!(x)) {                                               \
      std::printf("%s:%d: %s\n", __FILE__, __LINE__, #x);     \
      return 1;                                               \
    }                                                         \
  } while (0)

int main() {
  for (int64_t n : {0, 1, 2, 15, 16, 17, 1000}) {
    std::vector<std::atomic<int>> seen(static_cast<size_t>(n));
    for (auto& s : seen) s = 0;
    dfmm::parallel_for(n, [&](int64_t i) { ++seen[size_t(i)]; });
    for (auto& s : seen) CHECK(s == 1);
  }
  for (int64_t n : {1, 2, 1000})
    for (int64_t bad : {int64_t(0), n / 2, n - 1}) {
      bool caught = false;
      try {
        dfmm::parallel_for(n, [&](int64_t i) {
          if (i == bad) throw std::bad_alloc();
        });
      } catch (const std::bad_alloc&) {
        caught = true;
      }
      CHECK(caught);
    }
  int n = 0;
  try {  // of several, one
    dfmm::parallel_for(1000, [&](int64_t) { throw std::runtime_error("body"); });
  } catch (const std::runtime_error&) {
    ++n;
  }
  CHECK(n == 1);
  std::printf("parallel: ok\n");
  return 0;
}
