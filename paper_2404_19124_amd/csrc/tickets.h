// Host side of words that a kernel stores to pinned memory once it has read what stands beside them.
#pragma once
#include <chrono>
#include <cstdint>
#include <thread>

namespace specdraft {

// Waits until each of n words holds `ticket`: 0.  No other work is waited for, and nothing ends the wait but ask(), which is called
// every kTicketsAskMs and whose answer, if it is not 0, is returned (the device can no longer store them).
constexpr int kTicketsAskMs = 100;
template <typename Ask>
int wait_for_tickets(const uint32_t* words, int n, uint32_t ticket, Ask&& ask) {
  using clock = std::chrono::steady_clock;
  clock::time_point next{};
  int seen = 0;   // words that hold it
  for (int tries = 0;; ++tries) {
    while (seen < n && __atomic_load_n(words + seen, __ATOMIC_ACQUIRE) == ticket) ++seen;
    if (seen == n) return 0;
    if (tries < 1000) continue;   // (mostly they are there, or about to come)
    const clock::time_point now = clock::now();
    if (tries == 1000) next = now + std::chrono::milliseconds(kTicketsAskMs);
    if (now >= next) {
      next = now + std::chrono::milliseconds(kTicketsAskMs);
      if (const int answer = ask()) return answer;
    }
    std::this_thread::sleep_for(std::chrono::microseconds(10));
  }
}

}  // namespace specdraft
