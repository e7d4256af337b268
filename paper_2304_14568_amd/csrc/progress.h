// Reports of queued work that the host reads while the device goes on: one word
// of pinned memory per patient, the number of heads the patient has had << 1,
// the lowest bit set once it has stopped.  Host code only, without the runtime.
#pragma once
#include <cstdint>
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

}  // namespace admmbb
