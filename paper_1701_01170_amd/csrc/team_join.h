// How the workgroups of a launch agree on a team (k_dloop.h): those that run on one XCD
// register as members, everybody else is counted, and once all workgroups of the launch
// have registered the members run together.  A member that waits too long calls the
// team off for all.
//
// Both outcomes, the size and the members' places live in ONE 32-bit word, and every step
// below is one access to it, so that no member can act on an older state than another:
//   bits 0..15  workgroups registered
//   bits 16..30 members registered
//   bit 31      called off
// The team stands once the count is complete without bit 31.  Bit 31 is only ever set on
// an incomplete word (the compare-and-swap expects one), and a complete word does not
// change again; so every member decides from the same final word, its size included.
//
// Plain C++, so that the host can step through it as well.
#pragma once

#include <cstdint>

#if defined(__HIPCC__)
#define GR_TEAM_FN __host__ __device__ inline
#else
#define GR_TEAM_FN inline
#endif

namespace gr {

constexpr uint32_t kTeamOff = 1u << 31;
constexpr int kTeamMaxMembers = 255;  // the level barrier counts arrivals in 8 bits

// One workgroup's part.  Word: add(x) and cas(expected, x) return the word before,
// load() its value.
struct TeamJoin {
  enum Next : int { kRegister, kPoll, kCallOff, kDone };
  uint32_t grid;    // workgroups of the launch (< 65536)
  bool member;
  int polls;        // loads before a member calls the team off
  int next = kRegister;
  int index = -1;   // in the team (kDone: -1 = leave)
  int size = 0;     // of the team (kDone, index >= 0)
  bool called_off = false;  // by this workgroup
  uint32_t now = 0;

  GR_TEAM_FN TeamJoin(uint32_t g, bool m, int p) : grid(g), member(m), polls(p) {}

  // One access to the word.  A failed kCallOff means that the word has changed, which
  // happens at most once per workgroup of the launch and once for bit 31.
  template <class Word>
  GR_TEAM_FN void step(Word& w) {
    if (next == kRegister) {
      const uint32_t mine = member ? 0x10001u : 1u;
      const uint32_t old = w.add(mine);
      now = old + mine;
      index = member ? (int)(old >> 16 & 0x7fffu) : -1;
    } else if (next == kPoll) {
      now = w.load();
    } else {
      const uint32_t old = w.cas(now, now | kTeamOff);
      called_off = old == now;
      now = called_off ? now | kTeamOff : old;
    }
    if (!member || (now & kTeamOff)) {
      index = -1;
      next = kDone;
    } else if ((now & 0xffffu) == grid) {
      size = (int)(now >> 16);
      if (size > kTeamMaxMembers) index = -1;
      next = kDone;
    } else {
      next = polls-- > 0 ? kPoll : kCallOff;
    }
  }
};

}  // namespace gr
