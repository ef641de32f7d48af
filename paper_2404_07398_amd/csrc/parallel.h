// Host threads of the prepare phase.
#pragma once

#include <algorithm>
#include <cstdint>
#include <exception>
#include <thread>
#include <vector>

namespace ifl {

// f(0) .. f(count - 1), dealt in turn to at most 16 threads. The first
// exception of a thread is thrown here once all have ended; where no thread
// can be started, its share runs on this one.
template <typename F>
void parallel_for(int64_t count, const F& f) {
  const int nt = (int)std::min<int64_t>(count, std::max(1u, std::min(16u, std::thread::hardware_concurrency())));
  std::vector<std::exception_ptr> failed((size_t)std::max(nt, 1));
  auto share = [&](int t) {
    try {
      for (int64_t i = t; i < count; i += nt) f(i);
    } catch (...) {
      failed[(size_t)t] = std::current_exception();
    }
  };
  std::vector<std::thread> ts;
  ts.reserve((size_t)std::max(nt, 1));
  for (int t = 1; t < nt; ++t) {
    try {
      ts.emplace_back(share, t);
    } catch (...) {
      share(t);
    }
  }
  if (nt > 0) share(0);
  for (std::thread& t : ts) t.join();
  for (const std::exception_ptr& e : failed)
    if (e) std::rethrow_exception(e);
}

// Pieces that [0, n) is worth cutting into, and the start of piece p.
inline int64_t pieces_of(int64_t n) { return std::max<int64_t>(1, std::min<int64_t>(16, n / 4096)); }

}  // namespace ifl
