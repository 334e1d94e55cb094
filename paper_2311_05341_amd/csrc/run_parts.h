// Independent parts of the host's table building on threads.  Plain C++, no device code.
#pragma once

#include <exception>
#include <thread>

namespace dd {

constexpr int kMaxParts = 16;

// part(0) .. part(n - 1), n <= kMaxParts, at once where threads can be started (here, one after
// another, where not: no thread to be had, or no memory for its state).  Returns when all have
// returned; parts must not throw.
template <typename Part>
void run_parts(int n, const Part &part) {
  std::thread th[kMaxParts];
  for (int k = 1; k < n; ++k) try {
      th[k] = std::thread([&part, k] { part(k); });
    } catch (const std::exception &) {
      part(k);
    }
  part(0);
  for (std::thread &t : th)
    if (t.joinable()) t.join();
}

}  // namespace dd
