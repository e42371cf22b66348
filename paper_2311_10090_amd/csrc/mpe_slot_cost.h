// Host: whether a feed-forward rollout is faster in the slots of time that it holds (mpe_slots.h) than in one.  The unit of time is that
// in which 4, 8 and 12 wavefronts of a CU take 0.36, 0.56 and 0.81 for a step of the independent wavefronts (mpe_waves.h) while some CUs have
// none.  Measured, us, blocks of 4, 8, 12 on 64 to 192 CUs: 4 agents 4.8, 7.6, 10.9; 6 agents 5.3, 8.0, 11.2 (critic 9.5, 14.6, 20.3);
// 10 agents 7.9, 10.5, 15.4 (critic 12.0, 18.3, 27.2); medians over the batches of every shape lie within 10 %.  With a block of 8 or 12 on every CU the
// clock falls under the power limit and a step takes 12 to 25 % longer: 6 agents 5.4, 9.4, 13.9; waves_cost in mpe_waves.h, which compares
// full rounds, has the ratios of that.  The small-batch kernel's step is a table by 16-env blocks per CU, the kernels of up to 3 agents
// for full batches take 0.085 for every wavefront of 64 rows that their 64-env blocks put on a CU.  Measured on 4,542 batches (1 to 10
// agents and every predator-prey shape, 64 to 65,536 envs, 16 to 1,024 runs, both types, with and without critic, 50 to 128 steps), slots where
// this says so against one slot everywhere: 1.35 times as fast in the mean, 14 batches 2.5 to 7 % slower.  Slots wherever the size of
// the batch allows them: 397 slower, up to twice, above all where two or three slots of unequal length meet a chip that one slot fills.
#pragma once

#include "mpe_slots.h"

namespace mpe {

namespace {

// Up to how many envs the small-batch kernel is the faster one for a batch of whole runs (or of runs whose size suits the kernels
// for full batches), in tenths of 16-env blocks per CU.  Its time grows with every round of resident blocks, that of the
// others in steps; the lines are where the two measured curves cross, per shape.  128-step rollouts, us, this kernel
// against the others, at 16 x 256 x {1, 2, 3, 4, 6, 8, 12} envs (fp32 unless stated):
//   3 agents         193/418 295/419 411/531 493/537 727/958 953/945 1438/1339     (bf16 148/314 .. 537/675 744/681)
//   3 agents, critic 274/699 466/706 690/961 907/965 1549/1803 1975/1717 2812/2522
//   2 agents         176/390 281/388 296/393 322/394 543/527                       (critic 218/689 324/692 487/697 753/696)
//   1 agent          170/383 188/385 190/383 196/382 404/532 494/533 699/548
//   6 agents         364/661 674/670 942/1032 1248/1107                            (critic 537/1136 1039/1153 1523/1830 2011/1910)
//   tag (4,2,1)      221/626 356/644 545/640 852/638                               (critic 324/1109 604/1112 888/1119 1178/1124)
//   tag (10,3,2)     719/769 1381/1164
// `past`: where those kernels' first round of blocks (4 wavefronts of whole envs per CU) is just full, a second range.
struct SmallRange {
  uint32_t upto, past;
};
template <bool TAG, int N, bool AC, bool BF>
constexpr SmallRange small_range() {
  if constexpr (!TAG) {
    if constexpr (N == 1) return {80, 0};
    if constexpr (N == 2) return {AC ? 30 : 40, 0};
    if constexpr (N == 3) return {AC || BF ? 60 : 80, 0};
    constexpr SmallRange plain[7] = {{32, 0}, {23, 0}, {20, 30}, {17, 0}, {15, 0}, {12, 0}, {10, 0}};
    constexpr SmallRange critic[7] = {{35, 0}, {26, 40}, {22, 35}, {20, 32}, {16, 0}, {14, 21}, {12, 0}};
    return AC ? critic[N - 4] : plain[N - 4];
  } else {
    if constexpr (N == 2) return {AC ? 30 : 40, 0};
    if constexpr (N == 3) return {60, 0};
    if constexpr (N == 4) return {AC && BF ? 20 : 31, 0};
    if constexpr (N == 5) return AC && !BF ? SmallRange{24, 40} : SmallRange{22, 0};
    if constexpr (N == 6) return AC && !BF ? SmallRange{22, 35} : SmallRange{19, 30};
    if constexpr (N == 8) return {15, 0};
    return {AC ? 11 : 10, 0};
  }
}

// The same for a rollout in several slots of time (mpe_slots.h), whose envs are those of all slots; what it is measured
// against are the independent wavefronts (mpe_waves.h), of which a block per CU takes the same time whatever it holds.  128
// steps in five slots, us, this kernel against them, at 5 x {1,000, 2,048, 4,096, 8,192} envs (fp32 unless stated):
//   1 agent          43/133 44/133 63/135 133/136            critic 58/231 64/230 128/231 219/236     (bf16 31/92 31/93 44/93 83/94)
//   2 agents         60/129 63/128 91/129 186/188            critic 69/231 102/235 172/234 361/344    (bf16 45/93 48/94 72/94 151/132)
//   3 agents         65/137 88/138 135/143 239/222           critic 97/259 143/260 228/274 492/405    (bf16 51/96 68/96 100/98 193/142)
//   4 agents         75/151 114/152 189/215 400/323          critic 128/275 190/276 323/406 641/579
//   6 agents         134/160 188/178 314/257 607/515         critic 202/286 307/314 523/461 1044/883
//   10 agents        307/238 452/315 773/631                 critic 366/365 631/533 1253/1025
//   tag (4,2,1)      75/135 -/- 188/209 402/302              critic 124/247 -/- 322/376 639/542       (bf16 64/100 116/101 175/148 342/211)
//   tag (8,2,2)      180/164 270/229 458/340                 critic 282/288 423/407 719/619           (bf16 146/111 217/164 368/239)
template <bool TAG, int N, bool AC, bool BF>
constexpr SmallRange small_range_slots() {
  if constexpr (!TAG) {
    constexpr SmallRange plain[10] = {{105, 0}, {100, 0}, {85, 0}, {32, 52}, {22, 0}, {22, 30}, {15, 0}, {10, 0}, {10, 0}, {10, 0}};
    constexpr SmallRange critic[10] = {{110, 0}, {66, 0}, {75, 0}, {37, 52}, {26, 40}, {26, 38}, {20, 32}, {18, 27}, {11, 0}, {12, 0}};
    constexpr SmallRange plain_bf[3] = {{115, 0}, {63, 0}, {49, 0}}, critic_bf[3] = {{115, 0}, {61, 0}, {60, 0}};
    if constexpr (BF) return AC ? critic_bf[N - 1] : plain_bf[N - 1];
    else return AC ? critic[N - 1] : plain[N - 1];
  } else {
    // 2, 3, 4, 5, 6, 8, 10 agents
    constexpr SmallRange plain[7] = {{85, 0}, {72, 0}, {32, 52}, {22, 0}, {18, 0}, {10, 0}, {10, 0}};
    constexpr SmallRange critic[7] = {{61, 0}, {66, 0}, {37, 52}, {26, 0}, {24, 0}, {13, 0}, {10, 0}};
    constexpr SmallRange plain_bf[7] = {{62, 0}, {60, 0}, {21, 0}, {14, 0}, {11, 0}, {9, 0}, {10, 0}};
    constexpr SmallRange critic_bf[7] = {{58, 0}, {49, 0}, {27, 0}, {23, 0}, {16, 0}, {11, 0}, {10, 0}};
    constexpr int k = N <= 6 ? N - 2 : (N == 8 ? 5 : 6);
    return BF ? (AC ? critic_bf[k] : plain_bf[k]) : (AC ? critic[k] : plain[k]);
  }
}

struct BatchKind {
  int N;
  bool tag, bf, ac;
};

// A step of the small-batch kernel with `slots` of A's slots in flight.
inline float small_step(const BatchKind& k, const RolloutArgs& A, uint32_t slots) {
  struct Line { float at[4], more; };                  // 1, 2, 3, 4 blocks per CU, each one more
  static constexpr Line few[7] = {{{0.09f, 0.10f, 0.10f, 0.10f}, 0.055f}, {{0.12f, 0.195f, 0.195f, 0.21f}, 0.075f}, {{0.12f, 0.20f, 0.27f, 0.31f}, 0.095f},
                                  {{0.05f, 0.07f, 0.085f, 0.12f}, 0.030f}, {{0.07f, 0.11f, 0.17f, 0.25f}, 0.08f}, {{0.09f, 0.17f, 0.25f, 0.32f}, 0.09f},
                                  {{0.05f, 0.07f, 0.09f, 0.09f}, 0.04f}};
  static constexpr float plain[7][2] = {{0.12f, 0.08f}, {0.17f, 0.09f}, {0.19f, 0.14f}, {0.18f, 0.17f}, {0.22f, 0.21f}, {0.25f, 0.25f}, {0.28f, 0.12f}};
  static constexpr float critic[7][2] = {{0.095f, 0.095f}, {0.12f, 0.12f}, {0.16f, 0.15f}, {0.15f, 0.15f}, {0.20f, 0.20f}, {0.22f, 0.22f}, {0.26f, 0.26f}};
  const uint32_t cus = compute_units(), runs = A.TE / A.E;
  const uint32_t blocks = runs * ((A.E + 15) / 16) * slots, per_cu = blocks <= cus ? 1 : (blocks + cus - 1) / cus;
  if (k.N <= 3) {
    const Line& l = few[k.ac ? (k.N == 1 && k.bf ? 6 : 2 + k.N) : k.N - 1];
    return per_cu <= 4 ? l.at[per_cu - 1] : l.at[3] + l.more * float(per_cu - 4);
  }
  if (k.N == 6 || k.N == 8 || k.N == 10) {             // 8-env blocks while each has a CU
    const uint32_t eight = (A.TE + 7) / 8 * uint32_t(A.slots);
    static constexpr float alone[3][2] = {{0.11f, 0.09f}, {0.14f, 0.11f}, {0.18f, 0.13f}};
    const float one = alone[(k.N - 6) / 2][k.ac];
    if (eight <= cus) return one;
    if (k.N == 10 && k.ac) return one * float(((A.TE + 7) / 8 * slots + cus - 1) / cus);
  }
  const float* l = (k.ac ? critic : plain)[k.N - 4];
  return l[0] + l[1] * float(per_cu - 1);
}

// Steps of the first slot, the longest.
inline int32_t longest_slot(const RolloutArgs& A) { return A.slots > 1 ? A.T - (A.slots - 1) * A.span : A.T; }

inline bool equal_slots(const RolloutArgs& A) { return longest_slot(A) * 4 <= A.span * 5; }

// In the slots of A.  The blocks of slot 0 stay for its steps beyond a span, spread over the CUs.
inline float small_time(const BatchKind& k, const RolloutArgs& A) {
  if (A.slots <= 1) return small_step(k, A, 1) * float(A.T + 1);
  return small_step(k, A, uint32_t(A.slots)) * float(A.span + 1) + small_step(k, A, 1) * float(longest_slot(A) - A.span);
}

// Blocks of W independent wavefronts of which a CU holds `resident`, in the slots of A; one and a half steps to stage the weights.
inline float waves_time(int N, int W, int resident, const RolloutArgs& A) {
  auto step = [](uint32_t waves) { return waves == 0 ? 0.0f : (waves <= 4 ? 0.36f : (waves <= 8 ? 0.56f : 0.81f)); };
  const uint32_t runs = A.TE / A.E, eb = uint32_t(W) * (64u / uint32_t(N)), w = uint32_t(W);
  uint32_t cus = compute_units(), longs = runs * ((A.E + eb - 1) / eb), blocks = longs;
  bool stacked = false;
  if (A.slots > 1) {                                   // those of XCD 0, which has the most (spread_group)
    auto share = [](uint32_t n) { return n / 32u * 4u + (n % 32u < 4u ? n % 32u : 4u); };
    const uint32_t per_run = (A.E * uint32_t(A.slots) + eb - 1) / eb;
    // Blocks that share a CU are 32 apart on their XCD.  With 2, 4, .. blocks to a run, of which the first is long, they all have the same place
    // in their runs, until a second round mixes them (450 runs x 48 envs x 3 agents x 86 steps, critic, us, 883 in one slot, 962 in three).
    stacked = runs > 1 && !equal_slots(A) && 32 % per_run == 0 && runs * per_run < 2 * cus * uint32_t(resident);
    blocks = share(runs * per_run);
    longs = share(longs);
    cus = (cus + 7) / 8;
  }
  const uint32_t round = cus * uint32_t(resident), rest = blocks % round;
  const float a = float(longest_slot(A)) + 1.5f, b = stacked ? a : float(A.slots > 1 ? A.span : A.T) + 1.5f;
  if (blocks <= round) return step(w * ((blocks + cus - 1) / cus)) * b + step(w * ((longs + cus - 1) / cus)) * (a - b);
  const float full = step(w * uint32_t(resident)), all = makespan(round, longs, a, blocks - longs, b) * full;
  if (rest == 0) return all;
  // the last round by itself, with as many blocks on a CU as are left
  const uint32_t rounds = blocks - rest, first = longs < rounds ? longs : rounds;
  return fminf(all, makespan(round, first, a, rounds - first, b) * full + step(w * ((rest + cus - 1) / cus)) * (longs > rounds ? a : b));
}

// Whether one slot runs in the small-batch kernel.
inline bool small_in_one_slot(const BatchKind& k, const RolloutArgs& A, uint32_t upto) {
  const uint32_t runs = A.TE / A.E;
  return runs * ((A.E + 15) / 16) * 10 <= compute_units() * upto || (runs > 1 && A.E % 64 != 0 && k.N <= 3);
}
inline float one_slot_time(const BatchKind& k, RolloutArgs A, uint32_t upto) {
  A.slots = 1;
  const uint32_t cus = compute_units(), runs = A.TE / A.E;
  if (small_in_one_slot(k, A, upto)) {
    // runs of 32 envs: blocks of half-filled wavefronts beyond that kernel's range (1,024 runs x 3 agents 0.58)
    const bool halves = k.N <= 3 && runs > 1 && A.E % 32 == 0;
    return halves ? fminf(small_time(k, A), 0.048f * float(k.N) * float((A.TE / 32 + cus - 1) / cus) * float(A.T + 1)) : small_time(k, A);
  }
  const float waves = fminf(waves_time(k.N, 4, 3, A), fminf(waves_time(k.N, 8, 1, A), waves_time(k.N, 12, 1, A)));
  if (k.N > 3) return waves;
  const uint32_t blocks = runs * ((A.E + 63) / 64);
  const float time = 0.085f * float(k.N) * float((blocks + cus - 1) / cus) * float(A.T + 1);
  return k.N == 3 && !k.bf && !k.tag && A.TE == A.E ? fminf(time, waves) : time;
}

inline bool slots_pay(const RolloutArgs& A, float several, float one) { return several < (equal_slots(A) ? 0.95f : 0.90f) * one; }

}  // namespace

}  // namespace mpe
