// Reports of queued work that the host reads while the device goes on: one word
// of pinned memory per patient, the number of heads the patient has had << 1,
// the lowest bit set once it has stopped.  Host code only, without the runtime.
#pragma once
#include <chrono>
#include <cstdint>
#include <thread>
#include <vector>

namespace admmbb {

// The heads of one run.  They are counted from the words as the run finds them,
// the device being idle: a run that ended in an error after some of its heads
// were queued leaves nothing to be made up for in the next.
struct HeadCount {
  std::vector<uint32_t> base;  // per patient: heads before the run (31 bits)
  void begin(const volatile uint32_t* words, int patients) {
    base.resize(static_cast<size_t>(patients));
    for (int p = 0; p < patients; ++p) base[static_cast<size_t>(p)] = words[p] >> 1;
  }
  // whether `word` of patient p was written by the run's head number `heads`
  // (from 1) or a later one; counts wrap at 2^31
  bool reached(uint32_t word, int p, uint32_t heads) const {
    return (((word >> 1) - base[static_cast<size_t>(p)] - heads) & 0x7fffffffu) < 0x40000000u;
  }
};

// How the host waits for a report, as the process asked the runtime to wait for
// the device: by spinning (the runtime's default does the same), giving its turn
// to other threads in between, or asleep.  The last spins for as long as the
// runtime does before it blocks, then looks every 50 us: a few dense iterations
// are queued ahead of the one waited for, and a CG iteration takes longer.
enum class HostWait { spin, yield, sleep };

// Until reached(), or until dry() says that nothing is queued any more that could
// report; returns whether the report is there.
template <class Reached, class Dry>
bool wait_report(HostWait how, Reached reached, Dry dry) {
  using clock = std::chrono::steady_clock;
  constexpr std::chrono::microseconds kNap{50};
  const clock::time_point t0 = clock::now();
  for (uint32_t spins = 1; !reached(); ++spins) {
    if ((spins & 63u) == 0 && how == HostWait::yield) std::this_thread::yield();
    const bool nap = how == HostWait::sleep && (spins & 63u) == 0 && clock::now() - t0 > kNap;
    if (nap) {
      std::this_thread::sleep_for(kNap);
      spins |= 63u;  // once asleep, a look per nap
    }
    if ((nap || (spins & 0xfffu) == 0) && dry()) return reached();
  }
  return true;
}

}  // namespace admmbb
