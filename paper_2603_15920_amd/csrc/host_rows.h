// Row-independent host loops on a few threads.
#pragma once

#include <algorithm>
#include <exception>
#include <thread>
#include <vector>

namespace difvm {

// f(chunk, first, last) over consecutive chunks of n rows, at least per_thread rows each, on at most eight
// threads (the caller's among them).  Rows are independent, so what a row computes does not depend on
// the chunks.  The first exception of any chunk is rethrown here; where no thread can be started (the system refuses
// it, or the memory for its state) its chunk runs on the caller's: nothing may leave this function while
// threads run.
constexpr int MAX_CHUNKS = 8;
inline int n_chunks(int n, int per_thread) {
  int hw = (int)std::thread::hardware_concurrency();
  return std::max(1, std::min({n / per_thread, MAX_CHUNKS, hw > 0 ? hw : 1}));
}
template <class F>
void parallel_rows(int n, int per_thread, F&& f) {
  const int T = n_chunks(n, per_thread);
  std::exception_ptr err[MAX_CHUNKS];
  auto run = [&](int t) {
    try {
      f(t, (int)((long long)n * t / T), (int)((long long)n * (t + 1) / T));
    } catch (...) {
      err[t] = std::current_exception();
    }
  };
  std::vector<std::thread> th;
  th.reserve(T);
  int here[MAX_CHUNKS], n_here = 0;
  here[n_here++] = 0;
  for (int t = 1; t < T; ++t) {
    try {
      th.emplace_back(run, t);
    } catch (...) {
      here[n_here++] = t;
    }
  }
  for (int k = 0; k < n_here; ++k) run(here[k]);
  for (auto& x : th) x.join();
  for (int t = 0; t < T; ++t)
    if (err[t]) std::rethrow_exception(err[t]);
}

}  // namespace difvm
