// Waits of a wave for another wave of its own workgroup (a counter in LDS), in kernels whose workgroups wait for each other.
//
// What such a wave waits for may itself wait for other workgroups, by polls of memory that give up after SK_SPIN_LIMIT turns of 1 to 2 us.  A
// turn in here takes a tenth of a microsecond, so the same number of them would run out while the poll still succeeds, and its waves would go on
// without what they waited for.  So a wait in here ends when it is there or when a wave of the workgroup has said that it gave up; the bound behind that,
// some 128 times as many turns, is one that no poll reaches, and whoever reaches it says so as well.
#pragma once

namespace first {

constexpr unsigned SK_SPIN_LIMIT = 1u << 21;           // turns of a poll of memory
constexpr unsigned INSIDE_LIMIT = 1u << 28;            // turns of a wait inside a workgroup

enum class WaitEnd { THERE, GIVEN_UP, RAN_OUT };
// there(): what is waited for; given_up(): somebody of this workgroup did; pause(): between two looks.
template <typename There, typename GivenUp, typename Pause>
__attribute__((always_inline)) constexpr WaitEnd wait_inside(There there, GivenUp given_up, Pause pause) {
  for (unsigned turns = 0; turns < INSIDE_LIMIT; ++turns) {
    if (there()) return WaitEnd::THERE;
    if (given_up()) return WaitEnd::GIVEN_UP;
    pause();
  }
  return WaitEnd::RAN_OUT;
}

}  // namespace first
