// Internal: how the workgroups of a row count themselves (decode_short_impl.h).  Plain functions of what an atomic returned, so that
// every order of things can be gone through on the host as well (tests/short_count_model.cpp).
//
// A row has a 64-bit word in the device copy of the plan, zero between calls.  A workgroup whose state is in memory adds the step of its call,
// a number no other call has with a one in its low byte.  The word is `groups` steps for one workgroup, and only if it was zero and all
// workgroups of this call, and no others, have added: that one merges and puts the word back to zero.  A workgroup that finds anything but a
// number of steps of its own call (a call was aborted, another call uses this copy of the plan at the same time) puts the word back to zero and
// adds itself again.  Calls in turn are right whatever the word was.  Of two at once one may undo the count of the other, and a row of either
// may then never be merged: the first workgroup of a row makes it NaN, and its status one that is not zero, before it adds itself.
//
// The word only changes by these additions, from `groups` steps to zero, and from something that is no number of steps to zero: so an addition to
// what another call has left is wiped out before the workgroup that made it adds again, and none counts twice.
#pragma once
#include <cstdint>

namespace cocktail {

// The step of a call.  A call is named by the address of its dispatch packet: a slot in the ring of its queue, another one for every call and for
// every replay of a graph until the ring (16384 packets) comes round.  Mixed (the finalizer of SplitMix64; Steele, Lea, Flood 2014), so that
// sums of the steps of some calls are not those of another.
constexpr uint64_t short_step(uint64_t packet) {
  uint64_t x = (packet >> 6) * 0x9E3779B97F4A7C15ull;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  return (x ^ (x >> 31)) << 8 | 1u;
}
// Whether the word is a number of these steps (below 256: a row has 128 workgroups at most).
constexpr bool short_own(uint64_t word, uint64_t step) { return word == (word & 0xffu) * step; }
constexpr int kShortHealTries = 1024;   // (each of the other workgroups changes the word three times at most)

// Status of a row that has not been merged (not zero, whatever the number of its tokens is).
constexpr int32_t short_pending(int32_t expected) { return -expected - 1; }

}  // namespace cocktail
