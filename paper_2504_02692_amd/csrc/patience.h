// How long a workgroup waits for others of its launch (factor_roles.h).  Host code too, without HIP, so that a compiler without it can
// check the rule.
#pragma once
#ifdef __HIPCC__
#define GPTAQ_HOST_DEVICE __host__ __device__
#else
#define GPTAQ_HOST_DEVICE
#endif

namespace gptaq {

// A workgroup may have its place on the chip while others of its team have none yet, because kernels of other streams fill it: that ends
// when those kernels do, however long they take, so only time in which all of the team have started counts against a wait.  All of them
// running, a hand-over takes microseconds; it cannot fail unless something else writes into the workspace meanwhile.  Then the wait ends
// after a spell at whose beginning and end all had started, and in any case after kLongest spells, some two minutes.
struct Patience {
  static constexpr int kPolls = 1 << 20;           // a spell: some two seconds
  static constexpr int kLongest = 64;
  int polls = 0, spells = 0;
  bool together = false;
  // Whether a wait ends without what it waits for, asked after each poll; all_started() is asked once a spell.
  template <class AllStarted> GPTAQ_HOST_DEVICE bool over(AllStarted all_started) {
    if (++polls < kPolls) return false;
    polls = 0;
    const bool were = together;
    together = all_started();
    return (were && together) || ++spells == kLongest;
  }
};

}  // namespace gptaq
