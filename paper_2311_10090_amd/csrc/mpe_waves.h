// Fused rollout with independent wavefronts, for full batches: a wavefront owns WHOLE environments, as many as fit its
// 64 lanes (one lane per agent row; 60 to 64 of the lanes have a row), so the agents of an env never live in two
// wavefronts and nothing in the step loop waits for another wavefront.  A block is W such wavefronts around one staged
// copy of the weights.  Both scenarios; fp32 (split-operand) or bf16 networks of width 64; actor-critic (AC).
//
// A lane keeps its observation row in registers and stores it to the trajectory itself; the layer-1 operands and the
// logits travel between the row's lane and the matrix layout by 4 x 4 transposes between register index and 16-lane
// group (no memory).  LDS holds the weights and, per wavefront, the positions its agents exchange and the landmarks:
// 10 KB per wavefront less than with rows in LDS, which is what lets twelve wavefronts (three per SIMD, 168 registers
// each) share a CU in blocks of a size that suits the batch.
// What bounds it: vector issue and matrix time, as in mpe_policy_f32.hip: one wavefront per SIMD issues at the latency of
// its own chain; with two (20,011 envs x 6 agents, fp32) the vector unit is active for 79 % of the SIMD cycles and the matrix
// cores for 41 %, 39 % of which overlap.  Blocks of 64 envs with the rows in LDS, which these shapes used before, put 4 to 6
// wavefronts on a CU and met at a block barrier every step: that batch, 128 steps, mixed reward, 2,357 -> 1,233 us; predator-prey of 5 agents at 24,576 envs 2,124 -> 1,250 us.  (Looping over the pairs
// of tiles instead of unrolling them halves the code and changes nothing measurable.)  The arithmetic is that of the other
// kernels in the same order, and so are the results, bit for bit.
#pragma once

#include <type_traits>

#include "mpe_mlp64.h"
#include "mpe_scenario.h"
#include "mpe_slot_cost.h"

namespace mpe {

namespace {

template <int N_>
struct WaveSpread : SpreadScn<N_> {
  using Net = NetShape<6 * N_, 4 * N_ + 2>;
};
template <int N_, int L_, int G_>
struct WaveTag : TagScn<N_, L_, G_> {
  using Net = NetShape<TagScn<N_, L_, G_>::D, TagScn<N_, L_, G_>::D>;
};

// LDS of one wavefront: positions by step parity (the current one holds a new episode's after a reset), landmarks.
template <typename Scn>
struct WaveLds {
  static constexpr int N = Scn::N, EW = 64 / N, ROWS = EW * N;
  float4 xch[2][Scn::kTag ? ROWS : (ROWS + 1) / 2];    // predator-prey: position and velocity; else position (float2)
  float2 lm[EW * (Scn::L + 1)];
  float dmin[ROWS];
};

template <typename Scn, int W, bool AC, bool BF>
struct WavesSmem {
  using P = PkT<BF, Scn::Net::kWideIn, Scn::Net::kSlices1>;
  // staged image of a network: W1A, W2A, the part of W3A that is used, biases
  static constexpr size_t W3_BYTES = size_t(BF || Scn::Net::kRowTerms ? 2 : 6) * 64 * 16;
  static constexpr size_t OFF_BIAS = P::OFF_W3A + W3_BYTES, IMAGE = OFF_BIAS + P::BIAS_BYTES;
  static constexpr size_t OFF_CRITIC = IMAGE;
  static constexpr size_t OFF_WAVE = IMAGE * (AC ? 2 : 1);
  static constexpr size_t WAVE = (sizeof(WaveLds<Scn>) + 15) / 16 * 16;
  static constexpr size_t TOTAL = OFF_WAVE + W * WAVE;
  static_assert(IMAGE % 16 == 0 && TOTAL <= 160 * 1024, "LDS");
};

// Piece: SlotGrid for a launch of several slots of time (mpe_slots.h).  A run's envs are then E * slots, one slot's after the
// other's, and a lane has a slot of its own: wavefronts are full whatever the run size (runs of 16 envs x 3 agents in five
// slots take four wavefronts of 21 envs), and no two envs of a wavefront need their episodes end together.
template <typename Scn, int W, bool AC, bool BF, int MINW, typename Piece>
__global__ __launch_bounds__(W * 64, MINW) void rollout_waves_kernel(TagArgs TA, const uint8_t* __restrict__ packed,
                                                                     const uint8_t* __restrict__ packed_critic, Piece piece) {
  using M = WavesSmem<Scn, W, AC, BF>;
  using P = typename M::P;
  using Net = typename Scn::Net;
  using TS = typename Scn::Shape;
  constexpr bool kTag = Scn::kTag, SLOTS = kSlots<Piece>;
  constexpr int N = Scn::N, L = Scn::L, D = Scn::D, KIN = Net::KIN, KS1 = Net::kSlices1;
  constexpr int EW = 64 / N, EB = W * EW, ROWS = EW * N;
  constexpr int G = kTag ? TS::G : 1, NA = kTag ? TS::A : 0;
  constexpr bool kSpare = ROWS != 64;
  const RolloutArgs& A = TA.r;
  [[maybe_unused]] const TagPhys& tg = TA.tg;
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  WaveLds<Scn>& sm = *reinterpret_cast<WaveLds<Scn>*>(smem + M::OFF_WAVE + size_t(wave) * M::WAVE);
  const size_t TE = A.TE;
  uint32_t blk;
  if constexpr (SLOTS) {
    blk = spread_group(blockIdx.x);
    if (blk >= piece.groups) return;
  } else {
    blk = xcd_group(piece);
    if (blk >= piece.end) return;                        // whole block, before any barrier
  }
  // the blocks of a run are its own; its last one may be partly filled
  const uint32_t run_envs = SLOTS ? A.E * uint32_t(A.slots) : A.E;
  const uint32_t per_run = (run_envs + EB - 1) / EB, run = blk / per_run;
  const uint32_t env0 = (blk - run * per_run) * EB + wave * EW;        // first env of this wavefront inside its run
  const int nvalid = env0 < run_envs ? min(int(run_envs - env0), EW) : 0;
  const bool active = !kSpare || lane < ROWS;         // spare lanes shadow the wavefront's first row and store nothing
  const int row = active ? lane : 0, el = row / N, i = row - el * N;
  const bool in_range = el < nvalid, valid = active && in_range;
  uint32_t env = env0 + (in_range ? el : 0);
  uint32_t k_slot = 0;
  if constexpr (SLOTS) {
    k_slot = env / A.E;
    env -= k_slot * A.E;
  }
  const bool head = k_slot == 0;                      // the slot that reads and writes its env's state
  const size_t g = size_t(run) * A.E + (nvalid ? env : 0u);
  const int32_t max_ep = kTag ? tg.max_ep : A.ph.max_ep;

  // ---- weights of each network
  {
    auto stage = [&](const uint8_t* image, uint8_t* to) {
      const uint4* src = reinterpret_cast<const uint4*>(image + size_t(run) * P::RUN_BYTES);
      uint4* dst = reinterpret_cast<uint4*>(to);
      for (int k = threadIdx.x; k < int(M::OFF_BIAS / 16); k += W * 64) dst[k] = src[k];
      for (int k = threadIdx.x; k < int(P::BIAS_BYTES / 16); k += W * 64) dst[M::OFF_BIAS / 16 + k] = src[P::OFF_BIAS / 16 + k];
    };
    stage(packed, smem);
    if constexpr (AC) stage(packed_critic, smem + M::OFF_CRITIC);
  }
  const float* bias = reinterpret_cast<const float*>(smem + M::OFF_BIAS);
  [[maybe_unused]] const uint8_t* csm = smem + M::OFF_CRITIC;
  [[maybe_unused]] const float* cbias = reinterpret_cast<const float*>(csm + M::OFF_BIAS);

  // ---- this lane's agent; everything about the others is read from LDS where it is needed
  float px = 0.0f, py = 0.0f, vx = 0.0f, vy = 0.0f;
  int32_t ep = 0;
  uint32_t step = A.abs_step;
  // a new episode, keyed by the step that it starts at: every lane draws its own agent and landmarks i, i + N, ... of its env
  auto new_episode = [&](uint32_t start) {
    uint32_t env_r = env;
    asm volatile("" : "+v"(env_r));
    const uint4 d = philox4x32_10(env_r, start, uint32_t(i), kTagResetPos, A.seed, run);
    px = word_to_position(d.x);
    py = word_to_position(d.y);
    vx = vy = 0.0f;
    ep = 0;
#pragma unroll
    for (int k = 0; k < (L + N - 1) / N; ++k) {
      const int l = i + k * N;
      if (l < L) {
        const uint4 w = philox4x32_10(env_r, start, uint32_t(N + l), kTagResetPos, A.seed, run);
        float2 p = make_float2(word_to_position(w.x), word_to_position(w.y));
        if (kTag) { p.x *= 0.9f; p.y *= 0.9f; }        // obstacles start inside [-0.9, 0.9)
        if (active) sm.lm[el * (L + 1) + l] = p;
      }
    }
  };
  if (in_range) ep = A.st.ep_step[g];
  if (in_range && head) {      // the other slots of the env draw theirs; slot 0 may be writing these
    px = A.st.pos_a[(0 * N + i) * TE + g];
    py = A.st.pos_a[(1 * N + i) * TE + g];
    vx = A.st.vel_a[(0 * N + i) * TE + g];
    vy = A.st.vel_a[(1 * N + i) * TE + g];
  }
  [[maybe_unused]] int32_t ep0 = ep;
  [[maybe_unused]] TimeSlot slot = {0, A.T, 0, 0};
  int len = A.T;                                      // of the wavefront
  if constexpr (SLOTS) {
    counter_read(ep0);
    slot = time_slot(A.T, A.slots, A.span, int(k_slot), ep0, max_ep, true);
    if (!in_range) slot.len = 0;
    step += uint32_t(slot.t0);
    len = slot.len;
#pragma unroll
    for (int o = 32; o; o >>= 1) len = max(len, __shfl_xor(len, o));
    len = __builtin_amdgcn_readfirstlane(len);
  }
#pragma unroll
  for (int k = 0; k < (L + N - 1) / N; ++k) {         // landmarks i, i + N, ...
    const int l = i + k * N;
    if (l < L && active)
      sm.lm[el * (L + 1) + l] = in_range && head ? make_float2(A.st.pos_l[(0 * L + l) * TE + g], A.st.pos_l[(1 * L + l) * TE + g]) : make_float2(0.0f, 0.0f);
  }
  // what the lanes of an env read of each other, by step parity
  auto put = [&](int parity) {
    if (active) {
      if constexpr (kTag) sm.xch[parity][row] = make_float4(px, py, vx, vy);
      else reinterpret_cast<float2*>(sm.xch[parity])[row] = make_float2(px, py);
    }
  };
  auto pos = [&](int parity, int a) {                 // agent a of this lane's env
    if constexpr (kTag) {
      const float4 p = sm.xch[parity][el * N + a];
      return make_float2(p.x, p.y);
    } else {
      return reinterpret_cast<const float2*>(sm.xch[parity])[el * N + a];
    }
  };
  if (!head) new_episode(step);
  put(1);
  __syncthreads();   // weights staged; the only block-wide barrier
  // A wavefront past its run's last env ends here.  In this form, and not as a return, the rest of the kernel compiles as it
  // does without: the branch around the loop cost full batches 2 to 5 % (actor-critic, 32,768 envs x 6 agents 4.18 -> 4.40 ms).
  asm volatile("s_cmp_lg_u32 %0, 0\n\ts_cbranch_scc1 1f\n\ts_endpgm\n1:" : : "s"(nvalid) : "scc", "memory");
  [[maybe_unused]] TagRole me{};
  if constexpr (kTag) me = tag_role<TS>(i, tg);

  // The live entries of this lane's observation row; `cur`: where its env's positions are.
  auto build = [&](float (&o)[KIN], int cur) {
    float qx[N], qy[N], lx[L + 1], ly[L + 1], gvx[G], gvy[G];
    lx[L] = ly[L] = 0.0f;
    gvx[0] = gvy[0] = 0.0f;
#pragma unroll
    for (int a = 0; a < N; ++a) {
      if constexpr (kTag) {
        const float4 p = sm.xch[cur][el * N + a];
        qx[a] = p.x;
        qy[a] = p.y;
        if (a >= NA) {
          gvx[a - NA] = p.z;
          gvy[a - NA] = p.w;
        }
      } else {
        const float2 p = pos(cur, a);
        qx[a] = p.x;
        qy[a] = p.y;
      }
    }
#pragma unroll
    for (int k = 0; k < L; ++k) {
      const float2 p = sm.lm[el * (L + 1) + k];
      lx[k] = p.x;
      ly[k] = p.y;
    }
    agent_obs<Scn>(o, i, px, py, vx, vy, qx, qy, lx, ly, gvx, gvy);
  };
  auto store_row = [&](const float (&o)[KIN], float* dst, bool stores) {
    if (!stores) return;
    constexpr int CW = D % 4 == 0 ? 4 : 2;            // rows start on 16 bytes, or on 8
    typedef float vC __attribute__((ext_vector_type(CW)));
#pragma unroll
    for (int q = 0; q < D / CW; ++q) {
      vC v;
#pragma unroll
      for (int e = 0; e < CW; ++e) v[e] = CW * q + e < KIN ? o[CW * q + e < KIN ? CW * q + e : 0] : 0.0f;
      reinterpret_cast<vC*>(dst)[q] = v;
    }
  };
  // The networks on the wavefront's four tiles, two at a time.  z: the five logits of the lane's row; value: the critic's
  // output.  The critic runs on a pair of tiles just before the policy, so that both read one split of its inputs.
  auto forward = [&](const float (&o)[KIN], float (&z)[kNumActions], float& value, auto with_policy) {
    constexpr bool kPolicy = decltype(with_policy)::value;
    auto load_w3 = [&](const uint8_t* image) {
      W3Terms w;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const bf16x8* src = reinterpret_cast<const bf16x8*>(image + P::OFF_W3A) + lane;
        if constexpr (BF || Net::kRowTerms) {
          w.s[s].h = src[s * 64];
        } else {
          w.s[s].h = src[(s * 3 + 0) * 64];
          w.s[s].m = src[(s * 3 + 1) * 64];
          w.s[s].l = src[(s * 3 + 2) * 64];
        }
      }
      return w;
    };
    auto net = [&](const uint8_t* image, const float* b, const float (&tx)[KS1][8], const float (&ty)[KS1][8], f32x4& x, f32x4& y) {
      auto load = [&](int s, float (&vx)[8], float (&vy)[8]) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          vx[e] = tx[s][e];
          vy[e] = ty[s][e];
        }
      };
      if constexpr (BF) policy_core_bf<Net>(image, b, load_w3(image), load, x, y, lane);
      else policy_core<Net>(image, b, load_w3(image), tx, ty, x, y, lane);
    };
    constexpr bool kTerms = !BF && Net::kRowTerms;    // output layout of layer 3, see tile_logits in mpe_small.h
    uint32_t zs[4][4], cs[4];                         // [register][tile]
#pragma unroll
    for (int pr = 0; pr < 2; ++pr) {
      float tx[KS1][8], ty[KS1][8];
#pragma unroll
      for (int s = 0; s < KS1; ++s)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          uint32_t v[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int c = 32 * s + (Net::kWideIn ? 8 * q : 8 * (q & 1)) + e;
            v[q] = c < KIN ? __float_as_uint(o[c < KIN ? c : KIN - 1]) : 0u;
          }
          transpose_groups(v);
          tx[s][e] = __uint_as_float(v[2 * pr]);
          ty[s][e] = __uint_as_float(v[2 * pr + 1]);
        }
      f32x4 x, y;
      if constexpr (AC) {
        net(csm, cbias, tx, ty, x, y);
        cs[2 * pr] = __float_as_uint(kTerms ? (x[0] + x[1]) + x[2] : x[0]);
        cs[2 * pr + 1] = __float_as_uint(kTerms ? (y[0] + y[1]) + y[2] : y[0]);
      }
      if constexpr (kPolicy) {
        net(smem, bias, tx, ty, x, y);
        if constexpr (kTerms) {
          zs[0][2 * pr] = __float_as_uint((x[0] + x[1]) + x[2]);
          zs[0][2 * pr + 1] = __float_as_uint((y[0] + y[1]) + y[2]);
          zs[1][2 * pr] = __float_as_uint(x[3]);
          zs[1][2 * pr + 1] = __float_as_uint(y[3]);
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            zs[r][2 * pr] = __float_as_uint(x[r]);
            zs[r][2 * pr + 1] = __float_as_uint(y[r]);
          }
        }
      }
    }
    if constexpr (kPolicy) {
      transpose_groups(zs[0]);
      transpose_groups(zs[1]);
      if constexpr (kTerms) {
#pragma unroll
        for (int k = 0; k < 4; ++k) z[k] = __uint_as_float(zs[0][k]);
        z[4] = (__uint_as_float(zs[1][0]) + __uint_as_float(zs[1][1])) + __uint_as_float(zs[1][2]);
      } else {
        transpose_groups(zs[2]);
        transpose_groups(zs[3]);
#pragma unroll
        for (int k = 0; k < 4; ++k) z[k] = __uint_as_float(zs[k][0]);
        z[4] = __uint_as_float(zs[0][1]);
      }
    }
    if constexpr (AC) {
      transpose_groups(cs);
      value = __uint_as_float(cs[0]);
    }
  };

  float* obs_p = A.obs_traj;
  uint8_t* act_p = A.act_traj;
  float* rew_p = A.rew_traj;
  uint8_t* done_p = A.done_traj;
  [[maybe_unused]] float* logp_p = A.logp_traj;
  [[maybe_unused]] float* value_p = A.value_traj;
  // this lane's row and env in the time slices at the bases above, which go on a slice a step: in several slots with the
  // steps that it is ahead of the launch's first
  size_t row_off = g * N + i, env_off = g;
  const bool per_agent = kTag || A.ph.reward_mode == 1;
  [[maybe_unused]] uint32_t ticket = 0;
  auto ahead = [&](int32_t steps) {
    row_off += size_t(steps) * TE * N;
    env_off += size_t(steps) * TE;
  };
  if constexpr (SLOTS) {
    ahead(slot.t0);
    if (valid && i == 0) ticket = take_ticket(A, g);
  }
  float o[KIN];
#pragma unroll
  for (int c = 0; c < KIN; ++c) o[c] = 0.0f;
  wave_sync();
  build(o, 1);
  // state and last observation of the lanes that have run all their steps
  auto finish = [&]() {
    if (A.last_obs) store_row(o, A.last_obs + (g * N + i) * D, valid);
    if (valid) {
      A.st.pos_a[(0 * N + i) * TE + g] = px;
      A.st.pos_a[(1 * N + i) * TE + g] = py;
      A.st.vel_a[(0 * N + i) * TE + g] = vx;
      A.st.vel_a[(1 * N + i) * TE + g] = vy;
#pragma unroll
      for (int k = 0; k < (L + N - 1) / N; ++k) {
        const int l = i + k * N;
        if (l < L) {
          const float2 p = sm.lm[el * (L + 1) + l];
          A.st.pos_l[(0 * L + l) * TE + g] = p.x;
          A.st.pos_l[(1 * L + l) * TE + g] = p.y;
        }
      }
      if (i == 0 && !SLOTS) A.st.ep_step[g] = ep;
    }
  };
  for (int t = 0; t < len; ++t) {
    const int par = t & 1;
    const bool running = !SLOTS || t < slot.len, stores = valid && running, env_writer = stores && i == 0;
    const bool ended = SLOTS && head && t == slot.len;       // before the wavefront's other lanes
    if constexpr (SLOTS) {
      if (ended) finish();
    }
    if (obs_p) {
      store_row(o, obs_p + row_off * D, stores);
      obs_p += TE * (N * D);
    }
    float z[kNumActions], value = 0.0f;
    forward(o, z, value, std::true_type{});
    if constexpr (AC && SLOTS) {
      if (ended && valid && A.last_value) A.last_value[g * N + i] = value;
    }
    const uint32_t act = gumbel_argmax(z, A.seed, run, env, step, uint32_t(i));
    if (act_p) {
      if (stores) act_p[row_off] = uint8_t(act);
      act_p += TE * N;
    }
    if constexpr (AC) {
      // log pi(act | obs) = z_act - max - ln sum exp(z - max)
      float zmax = z[0], zact = z[0];
#pragma unroll
      for (int k = 1; k < kNumActions; ++k) {
        zmax = fmaxf(zmax, z[k]);
        zact = act == uint32_t(k) ? z[k] : zact;
      }
      float sum = 0.0f;
#pragma unroll
      for (int k = 0; k < kNumActions; ++k) sum += hw_exp2((z[k] - zmax) * kLog2e);
      if (logp_p) {
        if (stores) logp_p[row_off] = (zact - zmax) - kLn2 * hw_log2(sum);
        logp_p += TE * N;
      }
      if (value_p) {
        if (stores) value_p[row_off] = value;
        value_p += TE * N;
      }
    }

    // ---- transition on the positions of the step before (buffer par ^ 1)
    float qx[N], qy[N];
#pragma unroll
    for (int a = 0; a < N; ++a) {
      const float2 p = pos(par ^ 1, a);
      qx[a] = p.x;
      qy[a] = p.y;
    }
    if constexpr (kTag) {
      float lx[L + 1], ly[L + 1];
      lx[L] = ly[L] = 0.0f;
#pragma unroll
      for (int k = 0; k < L; ++k) {
        const float2 p = sm.lm[el * (L + 1) + k];
        lx[k] = p.x;
        ly[k] = p.y;
      }
      tag_move<TS>(act, i, me, tg, px, py, vx, vy, qx, qy, lx, ly);
    } else {
      agent_move<N>(act, i, A.ph, px, py, vx, vy, qx, qy);
    }
    put(par);
    wave_sync();
    if (rew_p) {
#pragma unroll
      for (int a = 0; a < N; ++a) {
        const float2 p = pos(par, a);
        qx[a] = p.x;
        qy[a] = p.y;
      }
      if constexpr (kTag) {
        const float r = tag_reward<TS>(i, me, tg, px, py, qx, qy);
        if (stores) rew_p[row_off] = r;
      } else {
        // coverage: this lane finds the distance of landmark i to the nearest agent; summed in landmark order
        const float2 mine = sm.lm[el * (L + 1) + i];
        float best2 = INFINITY;
#pragma unroll
        for (int a = 0; a < N; ++a) {
          const float dx = qx[a] - mine.x, dy = qy[a] - mine.y;
          best2 = fminf(best2, fmaf(dx, dx, dy * dy));
        }
        if (active) sm.dmin[row] = hw_sqrt(best2);
        wave_sync();
        float r = 0.0f;
#pragma unroll
        for (int a = 0; a < N; ++a) r -= sm.dmin[el * N + a];
        if (per_agent) {
          const float m = mixed_reward(r, overlap_count<N>(i, px, py, qx, qy, A.ph), A.ph);
          if (stores) rew_p[row_off] = m;
        } else if (env_writer) {
          rew_p[env_off] = r;
        }
      }
      rew_p += per_agent ? TE * N : TE;
    }
    ep += 1;
    const bool done = ep >= max_ep;
    if (done_p) {
      if (env_writer) done_p[env_off] = done ? 1 : 0;
      done_p += TE;
    }
    ++step;
    if constexpr (SLOTS) {
      if (t + 1 == slot.turn) {
        step += uint32_t(slot.jump);
        ahead(slot.jump);
      }
    }
    if (done) new_episode(step);
    wave_sync();               // the positions before a reset have been read
    if (done) put(par);
    wave_sync();
    build(o, par);
  }
  if constexpr (SLOTS) {
    if (valid && i == 0) settle_ticket(A, max_ep, g, ticket, ep0);
  }
  const bool ended = !SLOTS || (head && slot.len == len);
  if (ended) finish();
  if constexpr (AC) {
    if (A.last_value) {        // value of the observation after the last step
      float z[kNumActions], value = 0.0f;
      forward(o, z, value, std::false_type{});
      if (valid && ended) A.last_value[g * N + i] = value;
    }
  }
}

// Blocks of W wavefronts that share a CU: by LDS, and by registers (168 per wavefront up to 12 wavefronts, 256 up to 8).
template <typename Scn, int W, bool AC, bool BF>
struct WavesBlocks {
  static constexpr int EB = W * (64 / Scn::N);
  static constexpr size_t LDS = WavesSmem<Scn, W, AC, BF>::TOTAL;
  static constexpr int kResident = W != 4 || 2 * LDS > 160 * 1024 ? 1 : (3 * LDS > 160 * 1024 ? 2 : 3);
  static constexpr int kMinWaves = W * kResident > 8 ? 3 : 2;      // per SIMD, for the register budget
  static uint32_t count(const RolloutArgs& A) { return A.TE / A.E * ((A.E * uint32_t(A.slots) + EB - 1) / EB); }
};

// In the slots of A (SLOTS), or in one
template <typename Scn, int W, bool AC, bool BF, bool SLOTS>
hipError_t launch_waves_impl(const TagArgs& A, const void* packed, const void* critic, hipStream_t s) {
  using B = WavesBlocks<Scn, W, AC, BF>;
  auto kern = rollout_waves_kernel<Scn, W, AC, BF, B::kMinWaves, std::conditional_t<SLOTS, SlotGrid, GridPiece>>;
  static std::atomic<uint64_t> lds_allowed{0};
  if (hipError_t e = allow_lds(reinterpret_cast<const void*>(kern), B::LDS, lds_allowed); e != hipSuccess) return e;
  const uint32_t blocks = B::count(A.r);
  auto launch = [&](dim3 grid, auto piece) {
    hipLaunchKernelGGL(kern, grid, dim3(W * 64), B::LDS, s, A, static_cast<const uint8_t*>(packed), static_cast<const uint8_t*>(critic), piece);
  };
  if constexpr (SLOTS) {
    launch(spread_grid(blocks), SlotGrid{blocks});
    return hipGetLastError();
  } else {
    return launch_groups<W * 64>(blocks, launch);
  }
}

// Estimated time of a batch in blocks of W wavefronts, in steps of a CU with 12 resident wavefronts: full rounds of resident
// blocks, then a last one with as many blocks per CU as are left.  4, 8 and 12 wavefronts on every CU take 0.42,
// 0.75 and 1 (measured, 128 steps in one slot, us a step: 4 agents 4.8, 8.6, 12.6; 6 agents 5.4, 9.4, 13.9, critic 9.6, 16.3, 25.1; 10 agents 8.3,
// 12.6, 20.3; that is 0.38 to 0.41, 0.62 to 0.68 and 1; where some CUs have none, 8 and 12 are nearer to 4: mpe_slot_cost.h).  The estimate
// of that in the place of this one picks the same blocks to within 0.1 % of the time, but takes 20,011 envs x 6 agents out of their slots (1,234 us
// against 1,187).  12 with a critic or of 8 and more agents, with spilled registers, take 4 to 9 % more.  A block takes its steps and about one and a half more to stage the weights; in
// several slots slot 0, whose blocks come first, takes the longest.
template <typename Scn, int W, bool AC, bool BF>
float waves_cost(const RolloutArgs& A) {
  using B = WavesBlocks<Scn, W, AC, BF>;
  constexpr float kTwelve = !Scn::kTag && Scn::N > 8 ? 1.09f : (AC ? 1.07f : (!Scn::kTag && Scn::N == 8 ? 1.04f : 1.0f));
  const uint32_t cus = compute_units(), blocks = B::count(A), round = cus * B::kResident, rest = blocks % round;
  auto time_of = [](uint32_t waves) { return waves == 0 ? 0.0f : (waves <= 4 ? 0.42f : (waves <= 8 ? 0.75f : kTwelve)); };
  const float mean = float(A.T) / float(A.slots) + 1.5f, tail = blocks >= round ? float(A.slots > 1 ? A.span : A.T) + 1.5f : float(A.T - (A.slots - 1) * A.span) + 1.5f;
  return float(blocks / round) * time_of(W * B::kResident) * mean + time_of(W * ((rest + cus - 1) / cus)) * tail;
}

// The fewest steps of that estimate, and the W that takes them.  Where blocks of 4 and of
// 8 come out the same, 8 are faster by up to 14 % with fp32 weights: half the copies of them to stage, and no CU with one
// block of 4 beside one with two (8,192 / 24,576 envs x 10 agents 1,374 / 3,426 us against 1,580 / 3,820); with bf16 ones, a
// third of the bytes, 4 are (predator-prey, actor-critic, 12,288 envs x 6 agents 1,242 us against 1,280), and in several slots
// where the last round of 8 would be less than nine tenths full (16,384 envs x 1 agent 193 us against 209).
// Blocks of 12 only where three blocks of 4 don't fit a CU: those are as fast or up to 5 % faster than one of 12 (2 % slower in the worst
// of 58 batches of just under whole rounds).
struct WavesPlan {
  int W;
  float cost;
};
template <typename Scn, bool AC, bool BF>
constexpr bool kWavesTwelve = WavesBlocks<Scn, 4, AC, BF>::kResident < 3;
// One run of 3 agents of simple spread in one slot comes here up to 168 envs per CU: one block of 8 always
template <typename Scn, bool BF>
constexpr bool kWavesEightInOneSlot = !Scn::kTag && Scn::N == 3 && !BF;
template <typename Scn, bool AC, bool BF>
WavesPlan waves_plan(const RolloutArgs& A) {
  constexpr bool kTwelve = kWavesTwelve<Scn, AC, BF>;
  if (kWavesEightInOneSlot<Scn, BF> && A.slots == 1) return {8, waves_cost<Scn, 8, AC, BF>(A)};
  // slots of unequal length, which the estimate of whole rounds does not see
  if (A.slots > 1 && !equal_slots(A)) {
    const float t4 = waves_time(Scn::N, 4, WavesBlocks<Scn, 4, AC, BF>::kResident, A), t8 = waves_time(Scn::N, 8, 1, A), t12 = kTwelve ? waves_time(Scn::N, 12, 1, A) : INFINITY;
    if ((BF ? t4 <= t8 : t4 < t8) && t4 <= t12) return {4, t4};
    return t8 <= t12 ? WavesPlan{8, t8} : WavesPlan{12, t12};
  }
  const float c4 = waves_cost<Scn, 4, AC, BF>(A), c8 = waves_cost<Scn, 8, AC, BF>(A), c12 = kTwelve ? waves_cost<Scn, 12, AC, BF>(A) : INFINITY;
  const uint32_t cus = compute_units(), last8 = WavesBlocks<Scn, 8, AC, BF>::count(A) % cus;
  const bool four = BF || (A.slots > 1 && last8 && last8 * 10 < cus * 9);
  if ((four ? c4 <= c8 : c4 < c8) && c4 <= c12) return {4, c4};
  return c8 <= c12 ? WavesPlan{8, c8} : WavesPlan{12, c12};
}

template <typename Scn, bool AC, bool BF, bool SLOTS = false>
hipError_t launch_waves(const TagArgs& A, const void* packed, const void* critic, hipStream_t s) {
  [[maybe_unused]] const int W = waves_plan<Scn, AC, BF>(A.r).W;
  if constexpr (SLOTS || !kWavesEightInOneSlot<Scn, BF>) {
    if (W == 4) return launch_waves_impl<Scn, 4, AC, BF, SLOTS>(A, packed, critic, s);
    if constexpr (kWavesTwelve<Scn, AC, BF>) {
      if (W == 12) return launch_waves_impl<Scn, 12, AC, BF, SLOTS>(A, packed, critic, s);
    }
  }
  return launch_waves_impl<Scn, 8, AC, BF, SLOTS>(A, packed, critic, s);
}

// In the slots of A, where that pays: *taken.  With several runs, where a run's wavefronts and blocks are mostly full.
// `against`: that without slots this kernel would run, if not the small-batch kernel.  The same kernel either way: slots of equal length are compared in
// whole rounds (8 agents, critic, 20,011 envs 3,628 us in one slot, 3,737 in five; 6 agents, 20,011 envs 1,218 and 1,176), unequal ones taken from
// an estimated gain of 3 % on (10,000 envs x 5 agents x 74 steps 402 / 330 us); another kernel: from one of 5 and 10 % on.
template <typename Scn, bool AC, bool BF>
hipError_t launch_waves_slots(const TagArgs& A, bool against, const void* packed, const void* critic, hipStream_t s, bool* taken) {
  constexpr uint32_t EW = 64 / Scn::N, kUpto = small_range<Scn::kTag, Scn::N, AC, BF>().upto;
  constexpr BatchKind kind{Scn::N, Scn::kTag, BF, AC};
  const uint32_t envs = A.r.E * uint32_t(A.r.slots), waves = (envs + EW - 1) / EW;
  if (A.r.TE != A.r.E && (envs * 4 < waves * EW * 3 || waves * 4 < (waves + 3) / 4 * 4 * 3)) return hipSuccess;
  const WavesPlan plan = waves_plan<Scn, AC, BF>(A.r);
  RolloutArgs one = A.r;
  one.slots = 1;
  const bool same = against && !small_in_one_slot(kind, one, kUpto);
  if (same && equal_slots(A.r)) {
    if (plan.cost > 0.98f * waves_plan<Scn, AC, BF>(one).cost) return hipSuccess;
  } else {
    const float several = waves_time(Scn::N, plan.W, plan.W == 4 ? WavesBlocks<Scn, 4, AC, BF>::kResident : 1, A.r);
    const float single = one_slot_time(kind, one, kUpto);
    if (same ? several > 0.97f * single : !slots_pay(A.r, several, single)) return hipSuccess;
  }
  *taken = true;
  return launch_waves<Scn, AC, BF, true>(A, packed, critic, s);
}

}  // namespace

}  // namespace mpe
