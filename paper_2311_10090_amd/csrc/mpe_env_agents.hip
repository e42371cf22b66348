// Environment-only rollouts (seeded uniform actions) and single steps with one lane per AGENT, for both scenarios.
//
// A wavefront holds whole environments (as many as fit its 64 lanes, an even number so that its rows start on a
// 16-byte boundary of the trajectory), so the agents of an env exchange positions through LDS without a barrier.
//
// Rollout: a block is two wavefronts over the same envs.  Wave 0 steps them: move, exchange, next observation row into
// LDS.  Wave 1 does everything that does not depend on the state, one step AHEAD (the actions and the positions of an
// episode about to start come from the counter-based generator alone), and everything that leaves the chip, one step
// BEHIND (observation rows as contiguous 16-byte nontemporal stores, actions, rewards, done flags).  One block barrier
// per step; all exchanged data are double-buffered by step parity.
// What bounds it: small batches by the latency of a step, which is why the generator, the rewards and the stores are
// off wave 0's path and a lane carries one agent instead of a whole env; large ones by the trajectory writes.
#include "mpe_scenario.h"
#include "mpe_slots.h"

namespace mpe {

namespace {

// Envs per wavefront: the largest even number whose agents fit 64 lanes.
template <typename Scn>
constexpr int wave_envs() { return int(env_agents_block(Scn::N)); }

// What an agent passes to the others of its env: its new position, in predator-prey also its velocity.
template <bool TAG> struct Slot { float x, y; };
template <> struct __attribute__((aligned(16))) Slot<true> { float x, y, vx, vy; };
template <bool TAG>
__device__ __forceinline__ Slot<TAG> make_slot(float px, float py, float vx, float vy) {
  if constexpr (TAG) return {px, py, vx, vy};
  else return {px, py};
}

template <typename Scn>
struct AgentsSmem {
  static constexpr int N = Scn::N, L = Scn::L, EB = wave_envs<Scn>(), B = EB * N;
  static_assert(B <= 64 && (B * Scn::D) % 4 == 0, "whole 16-byte chunks");
  float obs[2][(B * Scn::D + 3) / 4 * 4];        // rows by step parity
  __attribute__((aligned(16))) Slot<Scn::kTag> xch[2][B];   // by step parity
  float2 fresh[2][EB * (N + L)];                 // positions of an episode that is about to start
  float dmin[B];                                 // coverage distances (4 and more agents)
  uint32_t act[2][B];
};

// Agent i's share of the coverage reward through LDS: the distance of landmark i (this lane's) to the nearest agent; the
// env's sum in landmark order, as coverage_reward forms it.  All lanes of the wavefront must come here.
template <int N>
__device__ __forceinline__ float coverage_by_lanes(float* dmin, int row, int el, bool has_row, float mylx, float myly,
                                                   const float (&qx)[N], const float (&qy)[N]) {
  float best2 = INFINITY;
#pragma unroll
  for (int a = 0; a < N; ++a) {
    const float dx = qx[a] - mylx, dy = qy[a] - myly;
    best2 = fminf(best2, fmaf(dx, dx, dy * dy));
  }
  wave_sync();
  if (has_row) dmin[row] = hw_sqrt(best2);
  wave_sync();
  float r = 0.0f;
#pragma unroll
  for (int a = 0; a < N; ++a) r -= dmin[el * N + a];
  return r;
}

// Entities i, i + N, ... of env el for the episode that starts at `step` (agents first, then landmarks).
template <typename Scn>
__device__ __forceinline__ void draw_fresh(float2* fresh, int el, int i, bool store, uint32_t env, uint32_t step, uint32_t seed, uint32_t run) {
  constexpr int N = Scn::N, ENT = Scn::N + Scn::L;
#pragma unroll
  for (int e = 0; e < (ENT + N - 1) / N; ++e) {
    const int ent = i + e * N;
    if (ent < ENT) {
      const uint4 d = philox4x32_10(env, step, uint32_t(ent), kTagResetPos, seed, run);
      float2 p = make_float2(word_to_position(d.x), word_to_position(d.y));
      if (Scn::kTag && e > 0) { p.x *= 0.9f; p.y *= 0.9f; }   // obstacles start inside [-0.9, 0.9)
      if (store) fresh[el * ENT + ent] = p;
    }
  }
}

// The groups of a launch that is not in pieces.  A form of its own, because the time of the step loops hangs on where
// their code lies: with a GridPiece for all, which moves it by 12 bytes, 8,192 envs x 6 agents of
// predator-prey took 134 instead of 117 us, 1,000 envs x 10 agents 138 instead of 129, 10,000 x 3 66.4 instead of 65.6.
struct WholeGrid {
  uint32_t end, per_xcd;
};
__device__ __forceinline__ uint32_t xcd_group(const WholeGrid& p) { return (blockIdx.x & 7u) * p.per_xcd + (blockIdx.x >> 3); }

template <typename Scn, typename Piece>
__global__ __launch_bounds__(128) void rollout_agents_kernel(TagArgs TA, Piece piece) {
  using M = AgentsSmem<Scn>;
  using TS = typename Scn::Shape;
  constexpr bool kTag = Scn::kTag, SLOTS = kSlots<Piece>;
  constexpr int N = Scn::N, L = Scn::L, D = Scn::D, EB = M::EB, B = M::B, ENT = N + L, LIVE = Scn::LIVE;
  constexpr int G = kTag ? TS::G : 1, NA = kTag ? TS::A : 0;
  __shared__ __attribute__((aligned(16))) M sm;
  const RolloutArgs& A = TA.r;
  [[maybe_unused]] const TagPhys& tg = TA.tg;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  const size_t TE = A.TE;
  int k_slot;
  uint32_t grp;
  if (!take_slot(A, piece, k_slot, grp)) return;
  const size_t g0 = size_t(grp) * EB;
  const int nvalid = TE - g0 < size_t(EB) ? int(TE - g0) : EB;
  const bool has_row = B == 64 || lane < B;                 // spare lanes shadow row 0 and store nothing
  const int row = has_row ? lane : 0, el = row / N, i = row - el * N;
  const size_t g = g0 + el;
  const bool in_range = g < TE, valid = has_row && in_range;
  const int32_t max_ep = kTag ? tg.max_ep : A.ph.max_ep;
  int32_t ep = in_range ? A.st.ep_step[g] : 0;
  const TimeSlot slot = group_slot<SLOTS>(A, k_slot, max_ep, g0, nvalid, lane);
  const bool head = k_slot == 0;                         // the slot that reads and writes the envs' state
  if (SLOTS) counter_read(ep);

  // the rows' trailing zeros are written once
  for (int k = threadIdx.x; k < int(sizeof(sm.obs) / 4); k += 128) (&sm.obs[0][0])[k] = 0.0f;
  __syncthreads();

  if (wave == 0) {
    // ================================================================ the envs
    float px = 0.0f, py = 0.0f, vx = 0.0f, vy = 0.0f;
    float qx[N], qy[N], lx[L + 1], ly[L + 1];
    [[maybe_unused]] float gvx[G], gvy[G];
    lx[L] = ly[L] = 0.0f;
    gvx[0] = gvy[0] = 0.0f;
    // a new episode's positions, drawn by the other wavefront
    auto take_fresh = [&](int parity) {
      const float2* f = &sm.fresh[parity][el * ENT];
#pragma unroll
      for (int a = 0; a < N; ++a) {
        qx[a] = f[a].x;
        qy[a] = f[a].y;
        if (a == i) { px = qx[a]; py = qy[a]; }
      }
#pragma unroll
      for (int k = 0; k < L; ++k) {
        lx[k] = f[N + k].x;
        ly[k] = f[N + k].y;
      }
    };
    if (!head) {
      __syncthreads();
      take_fresh(1);
      ep = 0;
    } else {
      if (in_range) {
        px = A.st.pos_a[(0 * N + i) * TE + g];
        py = A.st.pos_a[(1 * N + i) * TE + g];
        vx = A.st.vel_a[(0 * N + i) * TE + g];
        vy = A.st.vel_a[(1 * N + i) * TE + g];
      }
#pragma unroll
      for (int k = 0; k < L; ++k) {
        lx[k] = in_range ? A.st.pos_l[(0 * L + k) * TE + g] : 0.0f;
        ly[k] = in_range ? A.st.pos_l[(1 * L + k) * TE + g] : 0.0f;
      }
    }
    [[maybe_unused]] TagRole me{};
    if constexpr (kTag) me = tag_role<TS>(i, tg);
    auto exchange = [&](int parity) {   // this lane's new state out, its env's in
      if (has_row) sm.xch[parity][row] = make_slot<kTag>(px, py, vx, vy);
      wave_sync();
#pragma unroll
      for (int a = 0; a < N; ++a) {
        const Slot<kTag> p = sm.xch[parity][el * N + a];
        qx[a] = p.x;
        qy[a] = p.y;
        if constexpr (kTag) {
          if (a >= NA) {
            gvx[a - NA] = p.vx;
            gvy[a - NA] = p.vy;
          }
        }
      }
    };
    auto write_row = [&](int parity) {
      float o[LIVE];
#pragma unroll
      for (int c = 0; c < LIVE; ++c) o[c] = 0.0f;
      agent_obs<Scn>(o, i, px, py, vx, vy, qx, qy, lx, ly, gvx, gvy);
      if (has_row) {
        float2* dst = reinterpret_cast<float2*>(&sm.obs[parity][row * D]);
#pragma unroll
        for (int c = 0; c < LIVE / 2; ++c) dst[c] = make_float2(o[2 * c], o[2 * c + 1]);
      }
    };
    exchange(1);
    write_row(0);
    __syncthreads();
    for (int t = 0; t < slot.len; ++t) {
      const int par = t & 1;
      const uint32_t act = sm.act[par][row];
      if constexpr (kTag) tag_move<TS>(act, i, me, tg, px, py, vx, vy, qx, qy, lx, ly);
      else agent_move<N>(act, i, A.ph, px, py, vx, vy, qx, qy);
      exchange(par);
      ep += 1;
      if (ep >= max_ep) {
        take_fresh(par);
        if constexpr (kTag) {
#pragma unroll
          for (int k = 0; k < G; ++k) gvx[k] = gvy[k] = 0.0f;
        }
        vx = vy = 0.0f;
        ep = 0;
      }
      write_row(par ^ 1);
      __syncthreads();
    }
    if (valid && head) {
      A.st.pos_a[(0 * N + i) * TE + g] = px;
      A.st.pos_a[(1 * N + i) * TE + g] = py;
      A.st.vel_a[(0 * N + i) * TE + g] = vx;
      A.st.vel_a[(1 * N + i) * TE + g] = vy;
#pragma unroll
      for (int l = 0; l < L; ++l) {
        if (l % N == i) {
          A.st.pos_l[(0 * L + l) * TE + g] = lx[l];
          A.st.pos_l[(1 * L + l) * TE + g] = ly[l];
        }
      }
      if (i == 0 && !SLOTS) A.st.ep_step[g] = ep;
    }
  } else {
    // ================================================================ generator and stores
    const uint32_t gc = in_range ? uint32_t(g) : uint32_t(g0);
    const uint32_t run = gc / A.E, env = gc - run * A.E;
    const bool env_writer = valid && i == 0;
    const size_t row_off = size_t(gc) * N + i;
    const bool per_agent = kTag || A.ph.reward_mode == 1;
    // simple spread: the landmarks that the reward of a step is measured against (all of them for up to 3 agents,
    // landmark i for more)
    constexpr bool kByLanes = !kTag && N > 3;
    constexpr int RL = kTag ? 1 : (kByLanes ? 1 : L);
    [[maybe_unused]] float lx[RL], ly[RL];
    if constexpr (!kTag) {
#pragma unroll
      for (int k = 0; k < RL; ++k) {
        const int l = kByLanes ? i : k;
        lx[k] = head && in_range ? A.st.pos_l[(0 * L + l) * TE + g] : 0.0f;
        ly[k] = head && in_range ? A.st.pos_l[(1 * L + l) * TE + g] : 0.0f;
      }
    }
    [[maybe_unused]] TagRole me{};
    if constexpr (kTag) me = tag_role<TS>(i, tg);
    uint8_t* act_p = A.act_traj;
    float* rew_p = A.rew_traj;
    uint8_t* done_p = A.done_traj;
    float* obs_p = A.obs_traj;
    int t_draw = 0;                                          // local and absolute step of the next draw
    uint32_t step = A.abs_step + uint32_t(slot.t0);

    auto new_episode = [&](int parity) {                     // that starts at `step`
      uint32_t env_r = env;
      asm volatile("" : "+v"(env_r));
      draw_fresh<Scn>(sm.fresh[parity], el, i, has_row, env_r, step, A.seed, run);
    };
    auto take_landmarks = [&](int parity) {
      const float2* f = &sm.fresh[parity][el * ENT + N];
#pragma unroll
      for (int k = 0; k < RL; ++k) {
        const float2 p = f[kByLanes ? i : k];
        lx[k] = p.x;
        ly[k] = p.y;
      }
    };
    // action of step `step` and, if the env's episode ends with it, the next episode's positions; returns the latter
    auto draw = [&](int parity) {
      const uint32_t act = word_to_action(philox4x32_10(env, step, uint32_t(i), kTagUniformAction, A.seed, run).x);
      if (has_row) sm.act[parity][row] = act;
      if (act_p) {
        if (valid) act_p[row_off] = uint8_t(act);
        act_p += TE * N;
      }
      const bool done = ep + 1 >= max_ep, turn = ++t_draw == slot.turn;
      step += turn ? 1u + uint32_t(slot.jump) : 1u;
      if (turn && act_p) act_p += size_t(slot.jump) * TE * N;
      if (done) new_episode(parity);
      ep = done ? 0 : ep + 1;
      return done;
    };
    // reward and done flag of the step whose positions are in xch[parity]
    auto finish = [&](int parity, bool done) {
      if (rew_p) {
        float qx[N], qy[N], px = 0.0f, py = 0.0f;
#pragma unroll
        for (int a = 0; a < N; ++a) {
          const Slot<kTag> p = sm.xch[parity][el * N + a];
          qx[a] = p.x;
          qy[a] = p.y;
          if (a == i) { px = p.x; py = p.y; }
        }
        if constexpr (kTag) {
          const float r = tag_reward<TS>(i, me, tg, px, py, qx, qy);
          if (valid) rew_p[row_off] = r;
        } else {
          float r;
          if constexpr (kByLanes) r = coverage_by_lanes<N>(sm.dmin, row, el, has_row, lx[0], ly[0], qx, qy);
          else r = coverage_reward(qx, qy, lx, ly);
          if (per_agent) {
            const float m = mixed_reward(r, overlap_count<N>(i, px, py, qx, qy, A.ph), A.ph);
            if (valid) rew_p[row_off] = m;
          } else if (env_writer) {
            rew_p[gc] = r;
          }
        }
        rew_p += per_agent ? TE * N : TE;
      }
      if (done_p) {
        if (env_writer) done_p[gc] = done ? 1 : 0;
        done_p += TE;
      }
      if constexpr (!kTag) {
        if (done) take_landmarks(parity);
      }
    };
    auto flush = [&](int parity, float* slice) {
      float* dst = slice + g0 * (N * D);
      const bool vec4 = (reinterpret_cast<uintptr_t>(dst) & 15u) == 0;
      if (vec4 && nvalid == EB) stream_out_full<B * D / 4>(sm.obs[parity], dst, lane);
      else stream_out(sm.obs[parity], dst, nvalid * N * D, vec4, lane);
    };
    // time goes on: rewards and done flags are a step behind the rows, the actions a step ahead of them
    auto skip = [&](int steps) {
      if (rew_p) rew_p += size_t(steps) * TE * (per_agent ? N : 1);
      if (done_p) done_p += size_t(steps) * TE;
    };
    [[maybe_unused]] const int32_t ep0 = ep;
    if (!head) {
      skip(slot.t0);
      if (obs_p) obs_p += size_t(slot.t0) * TE * (N * D);
      if (act_p) act_p += size_t(slot.t0) * TE * N;
      ep = 0;
      new_episode(1);
      __syncthreads();
      if constexpr (!kTag) take_landmarks(1);
    }
    bool done_now = (!SLOTS || slot.len > 0) && draw(0), done_before = false;   // of steps t and t - 1
    __syncthreads();
    [[maybe_unused]] uint32_t ticket = 0;
    if (SLOTS && env_writer) ticket = take_ticket(A, g);
    for (int t = 0; t < slot.len; ++t) {
      const int par = t & 1;
      if (obs_p) {
        flush(par, obs_p);
        obs_p += TE * (N * D);
        if (t + 1 == slot.turn) obs_p += size_t(slot.jump) * TE * (N * D);
      }
      if (t > 0) {
        finish(par ^ 1, done_before);
        if (t == slot.turn) skip(slot.jump);
      }
      done_before = done_now;
      if (t + 1 < slot.len) done_now = draw(par ^ 1);
      __syncthreads();
    }
    if (!SLOTS || slot.len > 0) finish((slot.len - 1) & 1, done_before);
    if (A.last_obs && head) flush(slot.len & 1, A.last_obs);
    if (SLOTS && env_writer) settle_ticket(A, max_ep, g, ticket, ep0);
  }
}

// One transition under given actions.  Four wavefronts per block, each over envs of its own.
template <typename Scn>
struct StepSmem {
  static constexpr int N = Scn::N, L = Scn::L, EB = wave_envs<Scn>(), B = EB * N;
  float obs[(B * Scn::D + 3) / 4 * 4];
  __attribute__((aligned(16))) Slot<Scn::kTag> xch[B];
  float2 lm[EB * (L + 1)];
  float dmin[B];
  float2 fresh[EB * (N + L)];
};

constexpr int kStepWaves = 4;

template <typename Scn>
__global__ __launch_bounds__(kStepWaves * 64) void step_agents_kernel(TagArgs TA, uint32_t first) {
  using M = StepSmem<Scn>;
  using TS = typename Scn::Shape;
  constexpr bool kTag = Scn::kTag;
  constexpr int N = Scn::N, L = Scn::L, D = Scn::D, EB = M::EB, B = M::B, ENT = N + L, LIVE = Scn::LIVE;
  constexpr int G = kTag ? TS::G : 1, NA = kTag ? TS::A : 0;
  __shared__ __attribute__((aligned(16))) M all[kStepWaves];
  const RolloutArgs& A = TA.r;
  [[maybe_unused]] const TagPhys& tg = TA.tg;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  M& sm = all[wave];
  const size_t TE = A.TE;
  const size_t g0 = ((size_t(first) + blockIdx.x) * kStepWaves + wave) * EB;
  if (g0 >= TE) return;                                     // whole wavefront; there is no block barrier
  const int nvalid = TE - g0 < size_t(EB) ? int(TE - g0) : EB;
  const bool has_row = B == 64 || lane < B;
  const int row = has_row ? lane : 0, el = row / N, i = row - el * N;
  const bool in_range = g0 + el < TE, valid = has_row && in_range;
  const size_t g = in_range ? g0 + el : g0;
  const uint32_t run = uint32_t(g) / A.E, env = uint32_t(g) - run * A.E;
  const size_t row_off = g * N + i;
  const uint32_t given = TA.actions_in[row_off];
  float px = A.st.pos_a[(0 * N + i) * TE + g], py = A.st.pos_a[(1 * N + i) * TE + g];
  float vx = A.st.vel_a[(0 * N + i) * TE + g], vy = A.st.vel_a[(1 * N + i) * TE + g];
  int32_t ep = A.st.ep_step[g];
  const uint32_t act = given < uint32_t(kNumActions) ? given : 0u;
  // landmarks i, i + N, ... through LDS to the lanes of the env
#pragma unroll
  for (int k = 0; k < (L + N - 1) / N; ++k) {
    const int l = i + k * N;
    if (l < L && has_row) sm.lm[el * (L + 1) + l] = make_float2(A.st.pos_l[(0 * L + l) * TE + g], A.st.pos_l[(1 * L + l) * TE + g]);
  }
  if (LIVE < D) {
    for (int k = lane; k < int(sizeof(sm.obs) / 16); k += 64) reinterpret_cast<float4*>(sm.obs)[k] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  }
  if (has_row) sm.xch[row] = make_slot<kTag>(px, py, vx, vy);
  wave_sync();
  float qx[N], qy[N], lx[L + 1], ly[L + 1];
  [[maybe_unused]] float gvx[G], gvy[G];
  lx[L] = ly[L] = 0.0f;
  gvx[0] = gvy[0] = 0.0f;
  auto read_env = [&]() {
#pragma unroll
    for (int a = 0; a < N; ++a) {
      const Slot<kTag> p = sm.xch[el * N + a];
      qx[a] = p.x;
      qy[a] = p.y;
      if constexpr (kTag) {
        if (a >= NA) {
          gvx[a - NA] = p.vx;
          gvy[a - NA] = p.vy;
        }
      }
    }
  };
  read_env();
#pragma unroll
  for (int k = 0; k < L; ++k) {
    const float2 p = sm.lm[el * (L + 1) + k];
    lx[k] = p.x;
    ly[k] = p.y;
  }
  [[maybe_unused]] TagRole me{};
  if constexpr (kTag) {
    me = tag_role<TS>(i, tg);
    tag_move<TS>(act, i, me, tg, px, py, vx, vy, qx, qy, lx, ly);
  } else {
    agent_move<N>(act, i, A.ph, px, py, vx, vy, qx, qy);
  }
  wave_sync();
  if (has_row) sm.xch[row] = make_slot<kTag>(px, py, vx, vy);
  wave_sync();
  read_env();
  ep += 1;
  const bool done = ep >= (kTag ? tg.max_ep : A.ph.max_ep);
  if (A.rew_traj) {
    if constexpr (kTag) {
      const float r = tag_reward<TS>(i, me, tg, px, py, qx, qy);
      if (valid) A.rew_traj[row_off] = r;
    } else {
      float r;
      if constexpr (N > 3) {
        const float2 mine = sm.lm[el * (L + 1) + i];
        r = coverage_by_lanes<N>(sm.dmin, row, el, has_row, mine.x, mine.y, qx, qy);
      } else {
        r = coverage_reward(qx, qy, lx, ly);
      }
      if (A.ph.reward_mode == 1) {
        const float m = mixed_reward(r, overlap_count<N>(i, px, py, qx, qy, A.ph), A.ph);
        if (valid) A.rew_traj[row_off] = m;
      } else if (valid && i == 0) {
        A.rew_traj[g] = r;
      }
    }
  }
  if (A.done_traj && valid && i == 0) A.done_traj[g] = done ? 1 : 0;
  if (done) draw_fresh<Scn>(sm.fresh, el, i, has_row, env, A.abs_step + 1u, A.seed, run);
  wave_sync();
  if (done) {
    const float2* f = &sm.fresh[el * ENT];
#pragma unroll
    for (int a = 0; a < N; ++a) {
      qx[a] = f[a].x;
      qy[a] = f[a].y;
      if (a == i) { px = qx[a]; py = qy[a]; }
    }
#pragma unroll
    for (int k = 0; k < L; ++k) {
      lx[k] = f[N + k].x;
      ly[k] = f[N + k].y;
    }
    if constexpr (kTag) {
#pragma unroll
      for (int k = 0; k < G; ++k) gvx[k] = gvy[k] = 0.0f;
    }
    vx = vy = 0.0f;
    ep = 0;
  }
  if (valid) {
    A.st.pos_a[(0 * N + i) * TE + g] = px;
    A.st.pos_a[(1 * N + i) * TE + g] = py;
    A.st.vel_a[(0 * N + i) * TE + g] = vx;
    A.st.vel_a[(1 * N + i) * TE + g] = vy;
    if (i == 0) A.st.ep_step[g] = ep;
    if (done) {                                             // landmarks move at a reset only
#pragma unroll
      for (int l = 0; l < L; ++l) {
        if (l % N == i) {
          A.st.pos_l[(0 * L + l) * TE + g] = lx[l];
          A.st.pos_l[(1 * L + l) * TE + g] = ly[l];
        }
      }
    }
  }
  if (A.last_obs) {
    float o[LIVE];
#pragma unroll
    for (int c = 0; c < LIVE; ++c) o[c] = 0.0f;
    agent_obs<Scn>(o, i, px, py, vx, vy, qx, qy, lx, ly, gvx, gvy);
    if (has_row) {
      float2* dst = reinterpret_cast<float2*>(&sm.obs[row * D]);
#pragma unroll
      for (int c = 0; c < LIVE / 2; ++c) dst[c] = make_float2(o[2 * c], o[2 * c + 1]);
    }
    wave_sync();
    float* dst = A.last_obs + g0 * (N * D);
    const bool vec4 = (reinterpret_cast<uintptr_t>(dst) & 15u) == 0;
    if (vec4 && nvalid == EB) stream_out_full<B * D / 4>(sm.obs, dst, lane);
    else stream_out(sm.obs, dst, nvalid * N * D, vec4, lane);
  }
}

// Single steps: predator-prey, and simple spread from 4 agents (launch_step).
template <typename Scn>
hipError_t launch_agents(const TagArgs& A, hipStream_t s) {
  constexpr int EB = wave_envs<Scn>();
  const uint32_t waves = (A.r.TE + EB - 1) / EB;
  if (A.actions_in) {
    if constexpr (Scn::kTag || Scn::N > 3) {
      constexpr int kThreads = kStepWaves * 64;
      return launch_groups<kThreads>((waves + kStepWaves - 1) / kStepWaves, [&](dim3, const GridPiece& p) {
        hipLaunchKernelGGL(step_agents_kernel<Scn>, dim3(p.end - p.first), dim3(kThreads), 0, s, A, p.first);
      });
    } else {
      return hipErrorInvalidValue;
    }
  }
  if (A.r.slots > 1) {
    hipLaunchKernelGGL((rollout_agents_kernel<Scn, SlotGrid>), slots_grid(A.r, waves), dim3(128), 0, s, A, SlotGrid{waves});
    return hipGetLastError();
  }
  return launch_groups<128>(waves, [&](dim3 grid, const GridPiece& p) {
    if (p.first == 0 && p.end == waves) hipLaunchKernelGGL((rollout_agents_kernel<Scn, WholeGrid>), grid, dim3(128), 0, s, A, WholeGrid{p.end, p.per_xcd});
    else hipLaunchKernelGGL((rollout_agents_kernel<Scn, GridPiece>), grid, dim3(128), 0, s, A, p);
  });
}

}  // namespace

// Where the rollout above is faster than the kernels for large batches (mpe_env_kernels.hip, mpe_policy_wide.hip,
// mpe_tag.hip): while the latency of a step counts for more than the trajectory writes, for which those kernels own
// larger contiguous chunks.  Measured per 128-step rollout, us, this kernel against them:
//   3 agents    1,000 envs 82/117 (174 before, ragged)  10,000 90/120  16,384 95/119  32,768 233/153
//   4 agents    4,096 79/279   16,384 154/286   32,768 298/330
//   7 agents    4,096 107/552  12,288 383/557   20,000 619/819   32,768 1013/917
//   10 agents   4,096 259/793   8,192 541/793   12,288 759/809   16,384 990/866
//   tag (4,2,1) 1,000 80/135   16,384 105/140   65,536 435/449;  (10,3,2) 1,000 135/631  16,384 577/650  32,768 1096/1293
//   tag (6,2,2) 1,000 96/226    8,192 122/232   12,000 229/234   16,384 290/234
// One and two agents: one lane per env with its writer wavefront is as fast or faster throughout (44 against 68, 71
// against 68 us at 1,000 envs).
bool env_agents_faster(bool tag, int N, uint32_t TE) {
  const uint32_t per_cu = TE / compute_units();
  if (tag) {
    switch (N) {
      case 2: return per_cu < 128;
      case 3: return per_cu < 97;
      case 5: return per_cu < 52;
      case 6: return per_cu < 44;
      case 8: return per_cu < 40;
      default: return true;
    }
  }
  if (N <= 2) return false;
  if (N == 3) return per_cu <= 64;
  if (N == 4) return per_cu <= 128;
  return per_cu <= (N <= 7 ? 96 : 52);
}

// Slots of time for a rollout without a policy.  They pay while the latency of a step keeps the writes below what the
// trajectory's address pattern takes (5 to 5.5 TB/s), and cost up to 10 % beyond: TE envs write `bytes` a step, which takes
// about 0.26 N us with a lane per env (up to 3 agents of simple spread), 0.45 + 0.05 N us with a lane per agent.  Measured,
// 128 steps, us, 1 / 2 / 5 slots: 1 agent 1,000 envs 44 / 28 / 12, 32,768 40 / 26 / 23; 2 agents 16,384 65 / 43 / 43 (3.2
// TB/s with one slot), 24,576 71 / 59 / 60 (4.9), 32,768 72 / 78 / 79 (6.5); 3 agents 1,000 85 / 54 / 24, 12,288 96 / 71 / 66
// (3.5), 16,384 99 / 88 / 91 (4.7), 24,576 118 / 127 / 135 (7.1); 4 agents 4,096 76 / 49 / 41 (2.5), 8,192 77 / 78 / 83 (5.0);
// 5 agents 4,096 100 / 69 / 74 (3.5); 10 agents 1,000 145 / 91 / 67 (2.5), 2,048 120 / 132 / 135 (5.2); predator-prey of 4
// agents 1,000 85 / 54 / 22, 8,192 75 / 53 / 57 (3.5), 16,384 105 / 104 / 107 (7.0).
uint32_t env_slots(bool tag, int N, int D, uint32_t TE) {
  const bool per_env = !tag && N <= 3;
  const float rate = float(TE) * float(N * (4 * D + 1) + 5) / (per_env ? 0.26f * float(N) : 0.45f + 0.05f * float(N));   // bytes/us
  const float all = per_env ? 3.9e6f : 2.7e6f, two = per_env ? 4.95e6f : 4.8e6f, chip = float(compute_units()) / 256.0f;
  return rate <= all * chip ? ~0u : (rate <= two * chip ? 2u : 1u);
}

hipError_t launch_env_agents(bool tag, int N, int L, int G, const TagArgs& A, hipStream_t s) {
  if (tag) {
#define X(n, l, g) if (N == n && L == l && G == g) return launch_agents<TagScn<n, l, g>>(A, s);
    MPE_TAG_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
  }
  switch (N) {
    case 3: return launch_agents<SpreadScn<3>>(A, s);
    case 4: return launch_agents<SpreadScn<4>>(A, s);
    case 5: return launch_agents<SpreadScn<5>>(A, s);
    case 6: return launch_agents<SpreadScn<6>>(A, s);
    case 7: return launch_agents<SpreadScn<7>>(A, s);
    case 8: return launch_agents<SpreadScn<8>>(A, s);
    case 9: return launch_agents<SpreadScn<9>>(A, s);
    case 10: return launch_agents<SpreadScn<10>>(A, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace mpe
