// Random calls of timed launches against a simulated device whose clock runs
// on while the host asks for events: every launch's time must be the one it
// took, and no event may be handed out while a pending launch needs it.
// Prints "ok" and exits 0 on success.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <set>
#include <vector>

#include "timed_chain.hpp"

using phprng::bat::Pending;

struct Sim {
  std::mt19937_64 rng;
  std::vector<int64_t> at;  // completion time of each event's last record
  std::vector<int> free_events;
  std::vector<Pending<int>> pending;
  int64_t now = 0, device = 0, got = 0, expected = 0;
  size_t issued = 0, taken = 0;

  explicit Sim(uint64_t seed) : rng(seed) {}
  int take() {
    int e;
    if (free_events.empty()) {
      e = (int)at.size();
      at.push_back(0);
    } else {
      e = free_events.back();
      free_events.pop_back();
    }
    for (const auto &p : pending)
      if (p.a == e || p.b == e) {
        std::printf("event %d handed out while it is needed\n", e);
        std::exit(1);
      }
    return e;
  }
  void call(int launches) {
    device = std::max(device, now);
    int prev = take();
    at[prev] = device;
    for (int i = 0; i < launches; ++i) {
      const int64_t t = 1 + (int64_t)(rng() % 50);
      const int e = take();
      device += t;
      at[e] = device;
      expected += t;
      pending.push_back({i % 6, prev, e, i + 1 == launches});
      prev = e;
      ++issued;
    }
  }
  void sweep(bool wait) {
    phprng::bat::take_finished(
        pending,
        [&](int e) {
          now += (int64_t)(rng() % 30);  // the host is slow
          if (wait) now = std::max(now, at[e]);
          return at[e] <= now;
        },
        [&](const Pending<int> &p) {
          got += at[p.b] - at[p.a];
          ++taken;
        },
        [&](int e) { free_events.push_back(e); });
    if (std::set<int>(free_events.begin(), free_events.end()).size() != free_events.size()) {
      std::printf("an event was given back twice\n");
      std::exit(1);
    }
  }
};

int main() {
  for (uint64_t seed = 0; seed < 300; ++seed) {
    Sim s(seed);
    for (int step = 0; step < 200; ++step) {
      s.call(1 + (int)(s.rng() % 12));
      if (s.rng() % 3 == 0) s.sweep(false);
      if (s.rng() % 40 == 0) s.sweep(true);
    }
    s.sweep(true);
    if (!s.pending.empty() || s.got != s.expected || s.taken != s.issued ||
        s.free_events.size() != s.at.size()) {
      std::printf("seed %llu: time %lld of %lld, %zu of %zu launches, %zu of %zu events\n", (unsigned long long)seed,
                  (long long)s.got, (long long)s.expected, s.taken, s.issued, s.free_events.size(), s.at.size());
      return 1;
    }
  }
  std::puts("ok");
  return 0;
}
