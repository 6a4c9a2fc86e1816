// One wave on the host: 64 threads, each with its lane index; a ballot is a
// meeting of all of them.
#pragma once

#include <array>
#include <barrier>
#include <cstdint>
#include <functional>
#include <thread>
#include <vector>

namespace dc {

inline thread_local unsigned t_lane = 0;
inline std::barrier<> g_meet(64);
inline std::array<int, 64> g_votes;

// Runs fn on every lane and waits for all.
inline void run_wave(const std::function<void()>& fn) {
  std::vector<std::thread> lanes;
  for (unsigned i = 0; i < 64; ++i)
    lanes.emplace_back([&fn, i] {
      t_lane = i;
      fn();
    });
  for (std::thread& t : lanes) t.join();
}

}  // namespace dc

inline unsigned __lane_id() { return dc::t_lane; }
inline unsigned long long __ballot(int predicate) {
  dc::g_votes[dc::t_lane] = predicate;
  dc::g_meet.arrive_and_wait();
  unsigned long long b = 0;
  for (unsigned i = 0; i < 64; ++i) b |= static_cast<unsigned long long>(dc::g_votes[i] != 0) << i;
  dc::g_meet.arrive_and_wait();  // every lane has read before the next vote
  return b;
}
