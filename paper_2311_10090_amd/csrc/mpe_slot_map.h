// Which blocks and which steps the slots of time of a rollout take (mpe_slots.h).  Whole-number arithmetic, the same for host and device.
#pragma once

#include <cstdint>

namespace mpe {

// Blocks of one slot each.  One slot's groups come after the other's, slot 0, the longest, first.  Every XCD has an eighth of
// each slot's groups, in one piece (see xcd_group), the next eighth in the next slot: the XCDs' totals then differ by one, and
// 245 blocks that want a CU each are at most 31 on the 32 CUs of an XCD (in whole pieces 35 or none; with left-over
// blocks between them CUs stay idle beside others with two: 8,192 envs x 3 agents 353 against 215 us).
// k: 0 before; false: a block that is left over.  A walk over the slots before, which choose_slots keeps few.  A quotient in its place, together with
// four bytes more of arguments before A.slots, had the step loops spill other scalars (they spill 30 to 50): 4,096 envs x 3 agents x 128
// steps 132 -> 129 us, but predator-prey of 8 agents, bf16, 200 envs x 74 steps 85 -> 95.
constexpr bool slot_group(uint32_t block, uint32_t groups, int32_t slots, int& k, uint32_t& group) {
  uint32_t at = block >> 3;
  for (; k < slots; ++k) {
    const uint32_t c = (block + uint32_t(k)) & 7u, first = c * groups / 8u, n = (c + 1u) * groups / 8u - first;
    group = first + at;
    if (at < n) return true;
    at -= n;
  }
  return false;
}

// Blocks that have lanes of several slots: an XCD has every eighth piece of four neighbouring ones.
constexpr uint32_t spread_group(uint32_t block) {
  const uint32_t at = block >> 3;
  return (at >> 2) * 32u + (block & 7u) * 4u + (at & 3u);
}

struct TimeSlot {
  int32_t t0, len;     // first step, number of steps
  int32_t turn, jump;  // after `turn` steps time goes on `jump` steps later (turn 0: never)
};
// Slot k of `slots` of `span` steps, T >= slots * span.  ep: the env's episode counter; alike: whether it is that of every env that shares
// the slot (else slot 0 runs all steps).
constexpr TimeSlot time_slot(int32_t T, int32_t slots, int32_t span, int32_t k, int32_t ep, int32_t max_ep, bool alike) {
  if (!alike || ep < 0) return {0, k == 0 ? T : 0, 0, 0};
  const int32_t first = max_ep - ep > 1 ? max_ep - ep : 1, jump = (slots - 1) * span;
  if (k == 0) return {0, T - jump, first, jump};
  return {first + (k - 1) * span, span, 0, 0};
}

// In which blocks all envs have the same episode counter.  The counter changes from one env to the next at some envs, counted from the
// batch's first: blocks of b envs, from the first one on, are alike throughout exactly if b divides all of these, and so
// if it divides their greatest common divisor (0: they are all alike).  A counter below zero has all steps run in slot 0, as a change at 1 would.
constexpr uint32_t common_unit(uint32_t a, uint32_t b) {
  while (b) {
    const uint32_t rest = a % b;
    a = b;
    b = rest;
  }
  return a;
}
constexpr uint32_t counter_unit(uint32_t unit, uint32_t env, int32_t before, int32_t ep) {   // before: of the env before, or ep
  return unit == 1u ? 1u : (ep < 0 ? 1u : (before != ep ? common_unit(unit, env) : unit));
}

// The episode counter T steps later
constexpr int32_t counter_after(int32_t T, int32_t ep, int32_t max_ep) {
  const int64_t left = int64_t(max_ep) - ep, first = left > 1 ? left : 1;
  return T < first ? ep + T : int32_t((T - first) % max_ep);
}

}  // namespace mpe
