// A rollout in slots of time.  An episode starts from positions that the counter-based generator draws for (run, env,
// step of the start) and from nothing else, so the episodes of an env do not wait for each other: where a batch leaves the
// chip's SIMDs short of wavefronts, a rollout of T steps is launched as `slots` slots of `span` steps (whole episodes) that
// run side by side instead of one after the other.
//
// With `first` = steps until the env's current episode ends, slot k > 0 runs the steps [first + (k - 1) span, first + k span)
// from the draw of its first one.  Slot 0 runs what is left: the current episode, then a jump of (slots - 1) span steps and
// the steps up to T, so that it is the one slot that reads the env's state and the one that writes it, in that order.
// T >= slots * span, which keeps the jump inside the rollout whatever `first` is.  Work and results are those of one slot,
// bit for bit.
//
// The other slots read the episode counter alone, which has to stay until all of them have: every slot of an env takes
// a ticket after its read, and the last one to do so writes the counter's new value (a function of the old one and T) and
// puts the tickets back to zero.  No slot waits for another.
#pragma once

#include <cmath>

#include "mpe_launch.h"
#include "mpe_slot_map.h"

namespace mpe {

namespace {

// The groups of one slot in a launch of several.  A kernel instance takes this in the place of its other grids and is then
// one for slots: without them it has the code that it would have anyway (in one instance for both the step loops take up
// to 8 % longer, 129 envs x 6 agents x 39 steps without a policy 45.1 against 41.7 us).
struct SlotGrid {
  uint32_t groups;
};
template <typename Piece> constexpr bool kSlots = false;
template <> constexpr bool kSlots<SlotGrid> = true;

// The slot and the group of this block; false: a block that is left over.
template <typename Piece>
__device__ __forceinline__ bool take_slot(const RolloutArgs& A, const Piece& p, int& k, uint32_t& grp) {
  k = 0;
  if constexpr (!kSlots<Piece>) {
    grp = xcd_group(p);
    return grp < p.end;
  } else {
    return slot_group(blockIdx.x, p.groups, A.slots, k, grp);
  }
}

// The slot of a wavefront whose envs are [g0, g0 + n), n <= 64.
template <bool SLOTS>
__device__ __forceinline__ TimeSlot group_slot(const RolloutArgs& A, int k, int32_t max_ep, size_t g0, int n, int lane) {
  if constexpr (!SLOTS) return {0, A.T, 0, 0};
  const int32_t ep = A.st.ep_step[g0 + min(lane, n - 1)], ep0 = __builtin_amdgcn_readfirstlane(ep);
  TimeSlot s = time_slot(A.T, A.slots, A.span, k, ep0, max_ep, __ballot(ep != ep0) == 0ull);
  asm volatile("" : "+s"(s.len));   // the counters have been read when the wavefront comes to its next barrier
  return s;
}

// One lane per env takes its ticket once everything that shares the slot has read the counter (a block: behind a barrier
// that its wavefronts come to with the counters in registers, counter_read) and settles it at its end: nothing waits for the
// ticket before.  ep: the counter as read.
__device__ __forceinline__ void counter_read(int32_t& ep) { asm volatile("" : "+v"(ep)); }
__device__ __forceinline__ uint32_t take_ticket(const RolloutArgs& A, size_t g) {
  return __hip_atomic_fetch_add(A.st.tickets + g, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void settle_ticket(const RolloutArgs& A, int32_t max_ep, size_t g, uint32_t ticket, int32_t ep) {
  if (ticket != uint32_t(A.slots) - 1u) return;
  A.st.ep_step[g] = counter_after(A.T, ep, max_ep);
  A.st.tickets[g] = 0u;
}

}  // namespace

// Host: the most slots up to `want`, of whole episodes and at least kSlotSteps steps (what a block does before its first
// step, staging weights above all, takes as long as one to three of them).
// At most kMostSlots: every block walks over the slots before its own (512 envs x 3 agents without a policy, 2^20 steps, no outputs, 449 ms in 41,943 slots).
constexpr int32_t kSlotSteps = 16;
constexpr uint32_t kMostSlots = 256;
inline void choose_slots(RolloutArgs& A, int32_t max_ep, uint32_t want) {
  A.slots = 1;
  if (!A.st.tickets || want < 2 || max_ep > A.T / 2) return;
  if (uint64_t(A.TE) * uint64_t(A.T) > (1u << 30)) return;   // envs of all slots are counted in 32 bits
  const int32_t most = int32_t(want < kMostSlots ? want : kMostSlots), longer = A.T / (most + 1) + 1;   // the least span of no more than that
  const int64_t least = longer > kSlotSteps ? longer : kSlotSteps, span = (least + max_ep - 1) / max_ep * max_ep;
  if (2 * span > A.T) return;
  A.slots = int32_t(A.T / span);
  A.span = int32_t(span);
}

// Host: whether blocks of this many envs can have slots: a block whose envs have unlike counters runs all its steps in slot 0, in a
// block shape chosen for the shorter ones (128 steps, counters each its own, us, one slot against five: 3 agents 4,800 envs without a
// policy 96 / 166; 6 agents 1,000 envs 214 / 359, critic 290 / 504; recurrent, 3 agents 1,000 envs 321 / 726).  The wavefronts, whose lanes
// have a slot each, take any counters.
inline bool slots_fit(const RolloutArgs& A, uint32_t envs) { return A.alike % envs == 0; }

// Host: when the last of `longs` blocks of a steps and then `shorts` of b steps ends, each taken by the place for a block, of
// `places` on the chip, that is free first.
inline float makespan(uint32_t places, uint32_t longs, float a, uint32_t shorts, float b) {
  const uint32_t busy = longs % places, n[2] = {places - busy, busy};       // places that are free at free[0], free[1]
  float free[2] = {float(longs / places) * a, float(longs / places + 1) * a}, end = busy ? free[1] : free[0];
  if (const uint32_t rounds = shorts / places; rounds > 2) {
    for (float& f : free) f += float(rounds - 2) * b;
    shorts -= (rounds - 2) * places;
  }
  while (shorts) {
    const int k = n[1] && free[1] < free[0] ? 1 : 0;
    shorts -= shorts < n[k] ? shorts : n[k];
    free[k] += b;
    end = fmaxf(end, free[k]);
  }
  return end;
}

inline dim3 spread_grid(uint32_t blocks) { return dim3((blocks + 31) / 32 * 32); }   // see spread_group
// Blocks of a launch of several slots.
inline dim3 slots_grid(const RolloutArgs& A, uint32_t groups) { return dim3((groups * uint32_t(A.slots) + 7) / 8 * 8); }

}  // namespace mpe
