// mpe_slot_map.h against counting: every (slot, group) has one block, every step of an env one slot.  Prints the first difference and ends with 1.
#include <cstdio>
#include <vector>

#include "../paper_2311_10090_amd/csrc/mpe_slot_map.h"

namespace {

bool blocks(uint32_t groups, uint32_t slots) {
  std::vector<int> seen(size_t(groups) * slots, 0);
  uint32_t most = 0, least = ~0u;
  for (uint32_t x = 0; x < 8; ++x) {
    uint32_t mine = 0, before = 0;
    for (uint32_t b = x; b < (groups * slots + 7) / 8 * 8; b += 8) {
      int slot = 0;
      uint32_t group = 0;
      if (!mpe::slot_group(b, groups, int32_t(slots), slot, group)) continue;
      if (group >= groups || uint32_t(slot) >= slots || uint32_t(slot) < before) return std::printf("groups %u slots %u block %u\n", groups, slots, b), false;
      before = uint32_t(slot);                             // slot 0 first
      seen[size_t(slot) * groups + group] += 1;
      ++mine;
    }
    most = mine > most ? mine : most;
    least = mine < least ? mine : least;
  }
  for (int n : seen) if (n != 1) return std::printf("groups %u slots %u: a group with %d blocks\n", groups, slots, n), false;
  return most <= least + 1 || (std::printf("groups %u slots %u: XCDs of %u and %u blocks\n", groups, slots, least, most), false);
}

bool spread(uint32_t groups) {
  std::vector<int> seen(groups, 0);
  for (uint32_t b = 0; b < (groups + 31) / 32 * 32; ++b)
    if (const uint32_t g = mpe::spread_group(b); g < groups) seen[g] += 1;
  for (int n : seen) if (n != 1) return std::printf("spread %u\n", groups), false;
  return true;
}

bool steps(int32_t T, int32_t slots, int32_t span, int32_t ep, int32_t max_ep, bool alike) {
  std::vector<int> seen(T, 0);
  auto wrong = [&](const char* what) { return std::printf("T %d slots %d span %d ep %d max_ep %d: %s\n", T, slots, span, ep, max_ep, what), false; };
  int32_t after = ep;                                      // step by step
  std::vector<char> start(T + 1, 0);
  for (int32_t t = 0; t < T; ++t) {
    after += 1;
    if (after >= max_ep) { after = 0; start[t + 1] = 1; }
  }
  if (mpe::counter_after(T, ep, max_ep) != after) return wrong("counter");
  for (int32_t k = 0; k < slots; ++k) {
    const mpe::TimeSlot s = mpe::time_slot(T, slots, span, k, ep, max_ep, alike);
    if (k && s.len && !start[s.t0]) return wrong("a slot that does not start with an episode");
    int32_t t = s.t0;
    for (int32_t n = 0; n < s.len; ++n) {
      if (t < 0 || t >= T) return wrong("a step outside");
      seen[t] += 1;
      ++t;
      if (n + 1 == s.turn) {
        t += s.jump;
        if (t > T || !start[t]) return wrong("a jump into an episode");
      }
    }
    if (k == 0 && s.len && t != T) return wrong("slot 0 does not end with the rollout");
  }
  for (int n : seen) if (n != 1) return wrong("a step that is not run once");
  return true;
}

}  // namespace

bool alike(uint32_t seed) {
  // stretches of a length each, with a break here and there that is none, a counter below zero in some
  uint32_t state = seed * 2654435761u + 1u;
  auto draw = [&](uint32_t n) { state = state * 1664525u + 1013904223u; return (state >> 8) % n; };
  const uint32_t envs = 1 + draw(400), step = draw(3) ? 1 + draw(70) : envs;
  std::vector<int32_t> ep(envs);
  int32_t now = 3;
  for (uint32_t g = 0; g < envs; ++g) {
    if (g && g % step == 0) now = int32_t(draw(4));
    ep[g] = now;
  }
  if (draw(8) == 0) ep[draw(envs)] = -1;
  uint32_t unit = 0;
  for (uint32_t part = 0; part < 7; ++part) {              // strided, as threads do
    uint32_t mine = 0;
    for (uint32_t g = part; g < envs; g += 7) mine = mpe::counter_unit(mine, g, ep[g ? g - 1 : 0], ep[g]);
    unit = mpe::common_unit(unit, mine);
  }
  for (uint32_t block = 2; block <= 64; ++block) {
    bool all = true;
    for (uint32_t g = 0; g < envs; ++g) all = all && ep[g] >= 0 && ep[g] == ep[g / block * block];
    if (all != (unit % block == 0)) return std::printf("seed %u block %u unit %u\n", seed, block, unit), false;
  }
  return true;
}

int main() {
  for (uint32_t seed = 0; seed < 20000; ++seed) if (!alike(seed)) return 1;
  for (uint32_t groups = 1; groups <= 300; ++groups)
    for (uint32_t slots = 2; slots <= 41; ++slots) if (!blocks(groups, slots)) return 1;
  for (uint32_t groups : {1u, 7u, 8u, 41u, 1023u, 1024u, 40961u})
    for (uint32_t slots : {2u, 5u, 81u, 256u}) if (!blocks(groups, slots)) return 1;
  for (uint32_t groups = 1; groups <= 2000; ++groups) if (!spread(groups)) return 1;
  for (int32_t max_ep : {1, 2, 5, 16, 25, 40})
    for (int32_t span = max_ep; span <= 60; span += max_ep)
      for (int32_t slots : {2, 3, 5, 9})
        for (int32_t T = slots * span; T <= slots * span + 2 * max_ep + 1; ++T)
          for (int32_t ep = -3; ep <= max_ep + 3; ++ep) {
            if (!steps(T, slots, span, ep, max_ep, true) || !steps(T, slots, span, ep, max_ep, false)) return 1;
          }
  std::puts("slots ok");
  return 0;
}
