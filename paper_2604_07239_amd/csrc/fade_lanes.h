// fade_lanes.h — several host threads on one piece of work (host code only).
#pragma once
#include <thread>

// lane(0) on the caller's thread and lane(1) .. lane(n - 1) on threads of their own, n <= MAX; returns when all are done. Every lane takes
// work from a common pool until there is none, so where a thread cannot be started (no thread left, or no memory for its state)
// the others do it all: nothing is thrown past the threads that run.
template <int MAX, typename F> void fade_on_lanes(int n, F &&lane) noexcept {
  std::thread helpers[MAX];
  try {
    for (int l = 1; l < n && l < MAX; ++l) helpers[l] = std::thread([&lane, l] { lane(l); });
  } catch (...) {
  }
  lane(0);
  for (std::thread &t : helpers)
    if (t.joinable()) t.join();
}
