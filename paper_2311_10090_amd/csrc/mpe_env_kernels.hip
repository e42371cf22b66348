// Environment-only kernels with one lane per environment: reset, and, for 1 to 3 agents, single step and the persistent
// T-step rollout with seeded uniform actions (small batches of 3 agents, and more agents: mpe_env_agents.hip).  One
// lane owns one environment; the whole state of that env stays
// in registers for the T steps of a rollout and only the trajectory leaves the chip.
#include "mpe_slots.h"

namespace mpe {

namespace {

struct Lane {
  size_t g;       // global env index
  uint32_t run;   // g / E
  uint32_t env;   // g % E
  bool valid;
  size_t g0;      // first env of this wave
  int nvalid;     // number of valid envs in this wave
  int lane;
};

__device__ __forceinline__ Lane lane_info(uint32_t TE, uint32_t E) {
  Lane L;
  L.lane = threadIdx.x;
  L.g0 = size_t(blockIdx.x) * kWave;
  L.g = L.g0 + L.lane;
  L.valid = L.g < TE;
  const uint32_t gc = L.valid ? uint32_t(L.g) : 0u;
  L.run = gc / E;
  L.env = gc - L.run * E;
  const size_t left = size_t(TE) - L.g0;
  L.nvalid = left < size_t(kWave) ? int(left) : kWave;
  return L;
}

template <int N>
__global__ __launch_bounds__(kWave) void reset_kernel(StatePtrs st, uint32_t TE, uint32_t E,
                                                      uint32_t seed, float* __restrict__ obs) {
  __shared__ __attribute__((aligned(16))) float tile[ObsTile<N>::kFloats];
  const Lane L = lane_info(TE, E);
  Env<N> s;
  reset_env<N>(s, seed, L.run, L.env, 0u);
  if (L.valid) {
    store_state<N>(s, st, TE, L.g);
    if (st.tickets) st.tickets[L.g] = 0u;
  }
  if (obs) emit_obs<N>(s, tile, obs + L.g0 * (N * 6 * N), L.nvalid, L.lane);
}

__global__ __launch_bounds__(256) void read_counters_kernel(StatePtrs st, uint32_t TE, uint32_t* __restrict__ unit) {
  __shared__ uint32_t units[256];
  const uint32_t each = (TE + gridDim.x - 1) / gridDim.x, first = blockIdx.x * each, end = min(first + each, TE);   // each * gridDim.x < 2^32
  uint32_t q = 0;
  for (uint32_t g = first + threadIdx.x; g < end; g += 256) {
    const int32_t ep = st.ep_step[g];
    q = counter_unit(q, g, st.ep_step[g ? g - 1 : 0], ep);
    st.tickets[g] = 0u;
  }
  units[threadIdx.x] = q;
  __syncthreads();
  for (int n = 128; n; n >>= 1) {
    if (int(threadIdx.x) < n) units[threadIdx.x] = common_unit(units[threadIdx.x], units[threadIdx.x + n]);
    __syncthreads();
  }
  if (threadIdx.x == 0) unit[blockIdx.x] = units[0];
}

template <int N>
__global__ __launch_bounds__(kWave) void step_kernel(StatePtrs st, Phys ph, uint32_t TE, uint32_t E,
                                                     uint32_t seed, uint32_t abs_step,
                                                     const uint8_t* __restrict__ actions,
                                                     float* __restrict__ obs, float* __restrict__ reward,
                                                     uint8_t* __restrict__ done) {
  __shared__ __attribute__((aligned(16))) float tile[ObsTile<N>::kFloats];
  const Lane L = lane_info(TE, E);
  Env<N> s;
  uint32_t a[N];
  if (L.valid) {
    load_state<N>(s, st, TE, L.g);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const uint32_t v = actions[L.g * N + i];
      a[i] = v < uint32_t(kNumActions) ? v : 0u;
    }
  } else {
    zero_env<N>(s);
#pragma unroll
    for (int i = 0; i < N; ++i) a[i] = 0u;
  }
  bool d;
  if (ph.reward_mode == 1) {
    float r[N];
    transition<N, true>(s, a, ph, seed, L.run, L.env, abs_step, r, d);
    if (L.valid && reward) {
#pragma unroll
      for (int i = 0; i < N; ++i) reward[L.g * N + i] = r[i];
    }
  } else {
    float r[1];
    transition<N>(s, a, ph, seed, L.run, L.env, abs_step, r, d);
    if (L.valid && reward) reward[L.g] = r[0];
  }
  if (L.valid) {
    store_state<N>(s, st, TE, L.g);
    if (done) done[L.g] = d ? 1 : 0;
  }
  if (obs) emit_obs<N>(s, tile, obs + L.g0 * (N * 6 * N), L.nvalid, L.lane);
}

// --------------------------------------------------------------------------------------
// Wave-specialised persistent rollout for N <= 3.  A block is two wavefronts over the same 64 envs:
//   wave 0 (compute) keeps the 64 envs in registers, steps them, and drops each finished time
//           slice -- obs, reward, actions, done -- into one of two LDS slice buffers;
//   wave 1 (writer)  copies finished slices to HBM with 16-byte stores covering whole lines.
// The stores of a 1.9 GB trajectory back-pressure the issuing wave for most of a step; in a
// single wave that stall serialises with the arithmetic of the next step, here it overlaps.
// Two barriers per step hand the buffers back and forth:
//   X_t: writer has read slice t-1 out of buf[(t+1)&1]  -> compute may overwrite it
//   Y_t: compute has completed slice t in buf[t&1]       -> writer may read it
// Blocks are mapped to env groups XCD-aware: the hardware deals block b to XCD b % 8, so
// group = (b % 8) * groups_per_xcd + b / 8 gives each XCD one contiguous range of envs and
// the partial cache lines of neighbouring groups (actions: 192 B, done: 64 B per group and
// step) meet in the same L2 instead of being written back separately.
// --------------------------------------------------------------------------------------
template <int N, bool PER_AGENT>
struct SliceBuf {
  static constexpr int D = 6 * N;
  static constexpr int RW = PER_AGENT ? N : 1;         // rewards per env
  static constexpr int OBS_BYTES = kWave * N * D * 4;
  static constexpr int REW_OFF = OBS_BYTES;            // 64 * RW floats
  static constexpr int ACT_OFF = REW_OFF + kWave * 4 * RW;   // 64 * N bytes
  static constexpr int DONE_OFF = ACT_OFF + kWave * N; // 64 bytes
  static constexpr int BYTES = (DONE_OFF + kWave + 15) & ~15;
  static constexpr int OBS_F4 = OBS_BYTES / 16;
  static constexpr int FULL = OBS_F4 / kWave;          // full 64-lane rounds of obs
  static constexpr int TAIL = OBS_F4 % kWave;          // obs float4 left for the mixed round
  // lanes of the mixed round (the per-agent rewards have a round of their own)
  static constexpr int REW_L = TAIL, ACT_L = REW_L + (PER_AGENT ? 0 : 16), DONE_L = ACT_L + 4 * N, END_L = DONE_L + 4;
  static_assert(END_L <= kWave && 16 * RW <= kWave, "the rounds of the small outputs must fit one wavefront");
};

// PER_AGENT: the mixed reward, rew_traj is [T][TE][N].
// GENERAL: env counts that are no multiple of 64, or outputs whose time slices do not all start on 16 bytes: rows still
// leave in 16-byte pieces (a slice starts on 8 bytes), the small outputs element by element.  (128 steps of 1,000 envs x 1 agent 70 -> 45 us, 1,000 x 2 104 -> 72 us, 32,760
// x 3 206 -> 173 us against the one-wavefront kernel that such batches took before.)
// SLOTS: a launch of several slots of time (mpe_slots.h).
template <int N, bool GENERAL, bool PER_AGENT, bool SLOTS>
__global__ __launch_bounds__(2 * kWave) void rollout_uniform_ws_kernel(RolloutArgs A, uint32_t groups,
                                                                       uint32_t groups_per_xcd) {
  using SB = SliceBuf<N, PER_AGENT>;
  constexpr int RW = SB::RW;
  constexpr int D = 6 * N;
  __shared__ __attribute__((aligned(16))) uint8_t buf[2][SB::BYTES];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int k_slot = 0;
  uint32_t grp = (blockIdx.x & 7u) * groups_per_xcd + (blockIdx.x >> 3);
  if (SLOTS ? !take_slot(A, SlotGrid{groups}, k_slot, grp) : grp >= groups) return;  // whole block, before any barrier
  const size_t TE = A.TE;
  const size_t g0 = size_t(grp) * kWave;
  const TimeSlot slot = group_slot<SLOTS>(A, k_slot, A.ph.max_ep, g0, int(min(TE - g0, size_t(kWave))), lane);
  const bool head = k_slot == 0;              // the slot that reads and writes the envs' state

  if (wave == 0) {
    // ------------------------------------------------------------------ compute wave
    const bool valid = !GENERAL || g0 + lane < TE;
    const size_t g = valid ? g0 + lane : g0;      // lanes past the last env shadow the group's first and store nothing
    const uint32_t run = uint32_t(g) / A.E;
    const uint32_t env = uint32_t(g) - run * A.E;
    uint32_t step = A.abs_step + uint32_t(slot.t0);
    Env<N> s;
    [[maybe_unused]] int32_t ep0 = 0;
    [[maybe_unused]] uint32_t ticket = 0;
    if (head) load_state<N>(s, A.st, TE, g);
    else reset_env<N>(s, A.seed, run, env, step);
    if constexpr (SLOTS) {
      ep0 = head ? s.ep : A.st.ep_step[g];
      counter_read(ep0);
      __syncthreads();                           // the writer has read the counters
      if (valid) ticket = take_ticket(A, g);
    }
    auto write_obs = [&](uint8_t* b) {
      float2* row = reinterpret_cast<float2*>(b) + lane * (N * D / 2);
#pragma unroll
      for (int i = 0; i < N; ++i) build_agent_obs<N>(s, i, row + i * (D / 2));
    };
    write_obs(buf[0]);
    for (int t = 0; t < slot.len; ++t) {
      uint32_t a[N];
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const uint4 w = philox4x32_10(env, step, uint32_t(i), kTagUniformAction, A.seed, run);
        a[i] = word_to_action(w.x);
      }
      if (SLOTS && t + 1 == slot.turn) step += uint32_t(slot.jump);
      float r[RW];
      bool d;
      transition<N, PER_AGENT>(s, a, A.ph, A.seed, run, env, step, r, d);
      ++step;
      __syncthreads();  // X_t
      uint8_t* cur = buf[t & 1];
#pragma unroll
      for (int i = 0; i < RW; ++i) reinterpret_cast<float*>(cur + SB::REW_OFF)[lane * RW + i] = r[i];
#pragma unroll
      for (int i = 0; i < N; ++i) cur[SB::ACT_OFF + lane * N + i] = uint8_t(a[i]);
      cur[SB::DONE_OFF + lane] = d ? 1 : 0;
      write_obs(buf[(t + 1) & 1]);
      __syncthreads();  // Y_t
    }
    if (A.last_obs && head) {
      const float* last = reinterpret_cast<const float*>(buf[slot.len & 1]);
      if constexpr (GENERAL) stream_out(last, A.last_obs + g0 * (N * D), int(min(TE - g0, size_t(kWave))) * N * D, false, lane);
      else stream_out_full<SB::OBS_F4>(last, A.last_obs + g0 * (N * D), lane);
    }
    if (valid && head) store_state<N>(s, A.st, TE, g, !SLOTS);
    if (SLOTS && valid) settle_ticket(A, A.ph.max_ep, g, ticket, ep0);
  } else if constexpr (GENERAL) {
    // ------------------------------------------------------------------ writer wave, any size and alignment
    typedef float v4f_a8 __attribute__((ext_vector_type(4), aligned(8)));
    const int n = int(min(TE - g0, size_t(kWave)));          // envs of this group
    const int n4 = n * N * D / 4;                            // whole 16-byte pieces of their rows
    constexpr int kRounds = (SB::OBS_F4 + kWave - 1) / kWave;
    const size_t e0 = size_t(slot.t0) * TE + g0;             // the group's first env in its first time slice
    uint8_t* obs_g = A.obs_traj ? reinterpret_cast<uint8_t*>(A.obs_traj + e0 * (N * D)) : nullptr;
    uint8_t* act_g = A.act_traj ? A.act_traj + e0 * N : nullptr;
    float* rew_g = A.rew_traj ? A.rew_traj + e0 * RW : nullptr;
    uint8_t* done_g = A.done_traj ? A.done_traj + e0 : nullptr;
    v4f v[kRounds];
    v2f tail = {0.0f, 0.0f};
    float rew[RW];
    uint8_t act[N], done = 0;
    if (SLOTS) __syncthreads();
    for (int t = 0; t <= slot.len; ++t) {
      if (t > 0) {
        const size_t on = TE * (t == slot.turn ? 1u + size_t(slot.jump) : 1u);   // envs to the next time slice
        if (obs_g) {
#pragma unroll
          for (int k = 0; k < kRounds; ++k)
            if (k * kWave + lane < n4) __builtin_nontemporal_store(v[k], reinterpret_cast<v4f_a8*>(obs_g) + (k * kWave + lane));
          if ((n * N * D) % 4 && lane == 0) *reinterpret_cast<v2f*>(obs_g + size_t(n4) * 16) = tail;
          obs_g += on * (N * D) * 4;
        }
        if (rew_g) {
#pragma unroll
          for (int i = 0; i < RW; ++i)
            if (i * kWave + lane < n * RW) rew_g[i * kWave + lane] = rew[i];
          rew_g += on * RW;
        }
        if (act_g) {
#pragma unroll
          for (int i = 0; i < N; ++i)
            if (i * kWave + lane < n * N) act_g[i * kWave + lane] = act[i];
          act_g += on * N;
        }
        if (done_g) {
          if (lane < n) done_g[lane] = done;
          done_g += on;
        }
      }
      if (t == slot.len) break;
      __syncthreads();  // X_t
      __syncthreads();  // Y_t
      const uint8_t* cur = buf[t & 1];
      if (obs_g) {
#pragma unroll
        for (int k = 0; k < kRounds; ++k)
          if (k * kWave + lane < SB::OBS_F4) v[k] = *reinterpret_cast<const v4f*>(cur + (k * kWave + lane) * 16);
        if ((n * N * D) % 4) tail = *reinterpret_cast<const v2f*>(cur + n4 * 16);
      }
#pragma unroll
      for (int i = 0; i < RW; ++i) rew[i] = reinterpret_cast<const float*>(cur + SB::REW_OFF)[i * kWave + lane];
#pragma unroll
      for (int i = 0; i < N; ++i) act[i] = cur[SB::ACT_OFF + i * kWave + lane];
      done = cur[SB::DONE_OFF + lane];
    }
  } else {
    // ------------------------------------------------------------------ writer wave
    // Full rounds: lane l moves obs float4 number k*64 + l.  Mixed round: the obs tail, then
    // reward (16 lanes), actions (4N lanes) and done (4 lanes), one float4 each.
    const size_t e0 = size_t(slot.t0) * TE + g0;             // the group's first env in its first time slice
    uint8_t* obs_g = A.obs_traj ? reinterpret_cast<uint8_t*>(A.obs_traj + e0 * (N * D)) + lane * 16 : nullptr;
    const size_t obs_stride = TE * (N * D) * 4;
    int mix_lds = -1;          // byte offset inside a slice buffer, -1: lane idle in the mixed round
    uint8_t* mix_g = nullptr;
    size_t mix_stride = 0;
    if (lane < SB::TAIL) {
      if (A.obs_traj) {
        mix_lds = (SB::FULL * kWave + lane) * 16;
        mix_g = reinterpret_cast<uint8_t*>(A.obs_traj + e0 * (N * D)) + mix_lds;
        mix_stride = obs_stride;
      }
    } else if (lane < SB::ACT_L) {
      if (A.rew_traj) {
        mix_lds = SB::REW_OFF + (lane - SB::REW_L) * 16;
        mix_g = reinterpret_cast<uint8_t*>(A.rew_traj + e0) + (lane - SB::REW_L) * 16;
        mix_stride = TE * 4;
      }
    } else if (lane < SB::DONE_L) {
      if (A.act_traj) {
        mix_lds = SB::ACT_OFF + (lane - SB::ACT_L) * 16;
        mix_g = A.act_traj + e0 * N + (lane - SB::ACT_L) * 16;
        mix_stride = TE * N;
      }
    } else if (lane < SB::END_L) {
      if (A.done_traj) {
        mix_lds = SB::DONE_OFF + (lane - SB::DONE_L) * 16;
        mix_g = A.done_traj + e0 + (lane - SB::DONE_L) * 16;
        mix_stride = TE;
      }
    }
    v4f v[SB::FULL > 0 ? SB::FULL : 1];
    v4f vm = {0.0f, 0.0f, 0.0f, 0.0f};
    [[maybe_unused]] v4f vr = {0.0f, 0.0f, 0.0f, 0.0f};
    // the per-agent rewards' own round
    [[maybe_unused]] uint8_t* rew_g = PER_AGENT && A.rew_traj && lane < 16 * RW ? reinterpret_cast<uint8_t*>(A.rew_traj + e0 * RW) + lane * 16 : nullptr;
    if (SLOTS) __syncthreads();
    for (int t = 0; t <= slot.len; ++t) {
      if (t > 0) {
        if (obs_g) {
#pragma unroll
          for (int k = 0; k < SB::FULL; ++k) __builtin_nontemporal_store(v[k], reinterpret_cast<v4f*>(obs_g + k * (kWave * 16)));
          obs_g += obs_stride;
        }
        if (mix_lds >= 0) {
          *reinterpret_cast<v4f*>(mix_g) = vm;
          mix_g += mix_stride;
        }
        if constexpr (PER_AGENT) {
          if (rew_g) {
            *reinterpret_cast<v4f*>(rew_g) = vr;
            rew_g += TE * RW * 4;
          }
        }
        if (t == slot.turn) {
          if (obs_g) obs_g += size_t(slot.jump) * obs_stride;
          if (mix_lds >= 0) mix_g += size_t(slot.jump) * mix_stride;
          if (PER_AGENT && rew_g) rew_g += size_t(slot.jump) * TE * RW * 4;
        }
      }
      if (t == slot.len) break;
      __syncthreads();  // X_t
      __syncthreads();  // Y_t
      const uint8_t* cur = buf[t & 1];
      if (obs_g) {
#pragma unroll
        for (int k = 0; k < SB::FULL; ++k) v[k] = *reinterpret_cast<const v4f*>(cur + (k * kWave + lane) * 16);
      }
      if (mix_lds >= 0) vm = *reinterpret_cast<const v4f*>(cur + mix_lds);
      if constexpr (PER_AGENT) {
        if (rew_g) vr = *reinterpret_cast<const v4f*>(cur + SB::REW_OFF + lane * 16);
      }
    }
  }
}

inline dim3 env_grid(uint32_t TE) { return dim3((TE + kWave - 1) / kWave); }

inline bool aligned16p(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Whether the wave-specialised kernel can store whole waves and 16-byte pieces of every output.
template <int N>
inline bool ws_aligned(const RolloutArgs& A) {
  if (A.TE % kWave != 0) return false;
  if ((size_t(A.TE) * N) % 16 != 0) return false;  // action slices
  return aligned16p(A.obs_traj) && aligned16p(A.act_traj) && aligned16p(A.rew_traj) &&
         aligned16p(A.done_traj) && aligned16p(A.last_obs);
}

template <int N>
struct EnvLaunch {
  static hipError_t reset(const StatePtrs& st, uint32_t TE, uint32_t E, uint32_t seed, float* obs, hipStream_t s) {
    hipLaunchKernelGGL(reset_kernel<N>, env_grid(TE), dim3(kWave), 0, s, st, TE, E, seed, obs);
    return hipGetLastError();
  }
  static hipError_t step(const StatePtrs& st, const Phys& ph, uint32_t TE, uint32_t E, uint32_t seed,
                         uint32_t abs_step, const uint8_t* actions, float* obs, float* reward, uint8_t* done,
                         hipStream_t s) {
    hipLaunchKernelGGL(step_kernel<N>, env_grid(TE), dim3(kWave), 0, s, st, ph, TE, E, seed, abs_step,
                       actions, obs, reward, done);
    return hipGetLastError();
  }
  static hipError_t rollout(const RolloutArgs& A, hipStream_t s) {
    return A.slots > 1 ? rollout_slots<true>(A, s) : rollout_slots<false>(A, s);
  }
  template <bool SLOTS>
  static hipError_t rollout_slots(const RolloutArgs& A, hipStream_t s) {
    const uint32_t groups = (A.TE + kWave - 1) / kWave;
    const uint32_t per_xcd = (groups + 7) / 8;
    const dim3 grid = SLOTS ? slots_grid(A, groups) : dim3(per_xcd * 8), block(2 * kWave);
    const bool mixed = A.ph.reward_mode == 1;
    if (ws_aligned<N>(A)) {
      if (mixed) hipLaunchKernelGGL((rollout_uniform_ws_kernel<N, false, true, SLOTS>), grid, block, 0, s, A, groups, per_xcd);
      else hipLaunchKernelGGL((rollout_uniform_ws_kernel<N, false, false, SLOTS>), grid, block, 0, s, A, groups, per_xcd);
    } else {
      if (mixed) hipLaunchKernelGGL((rollout_uniform_ws_kernel<N, true, true, SLOTS>), grid, block, 0, s, A, groups, per_xcd);
      else hipLaunchKernelGGL((rollout_uniform_ws_kernel<N, true, false, SLOTS>), grid, block, 0, s, A, groups, per_xcd);
    }
    return hipGetLastError();
  }
};

}  // namespace

// `return CALL;` for the agent count; hipErrorInvalidValue for one that the kernel is not built for
#define MPE_CASE(N_, CALL) case N_: { constexpr int kN = N_; return CALL; }
// step and rollout of the lane-per-env kernels: up to 3 agents
#define MPE_DISPATCH_FEW(N_, CALL) \
  switch (N_) { MPE_CASE(1, CALL) MPE_CASE(2, CALL) MPE_CASE(3, CALL) default: return hipErrorInvalidValue; }
#define MPE_DISPATCH_N(N_, CALL)                                                               \
  switch (N_) {                                                                                \
    MPE_CASE(1, CALL) MPE_CASE(2, CALL) MPE_CASE(3, CALL) MPE_CASE(4, CALL) MPE_CASE(5, CALL)  \
    MPE_CASE(6, CALL) MPE_CASE(7, CALL) MPE_CASE(8, CALL) MPE_CASE(9, CALL) MPE_CASE(10, CALL) \
    default: return hipErrorInvalidValue;                                                      \
  }

hipError_t launch_reset(int N, const StatePtrs& st, uint32_t TE, uint32_t E, uint32_t seed, float* obs,
                        hipStream_t s) {
  MPE_DISPATCH_N(N, EnvLaunch<kN>::reset(st, TE, E, seed, obs, s));
}

hipError_t launch_read_counters(const StatePtrs& st, uint32_t TE, uint32_t* unit, hipStream_t s) {
  hipLaunchKernelGGL(read_counters_kernel, dim3(counter_blocks(TE)), dim3(256), 0, s, st, TE, unit);
  return hipGetLastError();
}

hipError_t launch_step(int N, const StatePtrs& st, const Phys& ph, uint32_t TE, uint32_t E, uint32_t seed,
                       uint32_t abs_step, const uint8_t* actions, float* obs, float* reward, uint8_t* done,
                       hipStream_t s) {
  // One lane per env up to 3 agents (65,536 envs x 3 agents 5.4 us, 6.7 us with one lane per agent); for more agents
  // one lane per agent (4 / 7 / 10 agents at 8,192 envs: 4.3 -> 3.8, 15.3 -> 5.2, 14.3 -> 8.2 us).
  if (N <= 3) MPE_DISPATCH_FEW(N, EnvLaunch<kN>::step(st, ph, TE, E, seed, abs_step, actions, obs, reward, done, s));
  TagArgs A{};
  A.r.st = st;
  A.r.ph = ph;
  A.r.TE = TE;
  A.r.E = E;
  A.r.seed = seed;
  A.r.abs_step = abs_step;
  A.r.T = 1;
  A.r.rew_traj = reward;
  A.r.done_traj = done;
  A.r.last_obs = obs;
  A.actions_in = actions;
  return launch_env_agents(false, N, N, 0, A, s);
}

hipError_t launch_rollout_uniform(int N, const RolloutArgs& A, hipStream_t s) {
  RolloutArgs B = A;
  choose_slots(B, A.ph.max_ep, env_slots(false, N, 6 * N, A.TE));
  auto by_agents = [&]() { return env_agents_faster(false, N, B.work()) || (N > 3 && B.slots > 1); };
  if (!slots_fit(B, by_agents() ? env_agents_block(N) : kWave)) B.slots = 1;
  if (by_agents()) {
    TagArgs TA{};
    TA.r = B;
    return launch_env_agents(false, N, N, 0, TA, s);
  }
  // many agents: one lane per agent (the wide fused kernel without its policy) writes contiguous pieces of the
  // trajectory
  if (N > 3) return launch_rollout_uniform_wide(N, A, s);
  MPE_DISPATCH_FEW(N, EnvLaunch<kN>::rollout(B, s));
}

}  // namespace mpe
