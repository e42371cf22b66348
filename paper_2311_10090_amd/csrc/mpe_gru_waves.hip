// Fused rollout with the recurrent policy for full batches of one run: a wavefront owns WHOLE environments, as many as
// fit 32 agent rows, and evaluates the whole network on them, so nothing in the step loop waits for another wavefront.
// (mpe_policy_gru.hip keeps the weights of 16 units in each wavefront's registers and passes the rows' activations through
// LDS, with seven block barriers a step; small batches and several runs stay there.)
//
// Rows are stationary here and weights move: the carried state (fp32, 64 registers), its bf16 copy and the activations
// never leave the registers of their wavefront, because the rows of every weight operand are permuted so that the
// accumulators of one layer are the B operands of the next (GruWavePk::unit).  A block is 8 wavefronts, two per SIMD, around
// 144 KB of LDS that hold three quarters of the gates' operands; the other quarter and the small layers (92 KB, 124 KB with
// the critic) are read from the L2 each step.  Both come through short rings of operands in flight, and every pair of matrix
// instructions is followed by a piece of another tile's activation, so that one wavefront's matrix and vector work are in
// flight together: sched_barrier fences keep that order.  Both halves of a wavefront hold the same 32
// agent rows in the environment's part; each draws one of the two blocks of sampling noise.
//
// What bounds it: issue and power.  A step of a wavefront issues 16,100 SIMD cycles with the critic (4,300 of them for 536
// matrix instructions, 8 of each one's 16 cycles; 6,300 for 790 exp and rcp), and the two wavefronts of a SIMD take 42,900 cycles a step:
// an instruction is issued in 86 % of them, the vector unit active in 73 %, the matrix cores busy in 40 %, a third of that at the same
// time.  The clock is 1.8 to 2.0 GHz: matrix instructions on real data run against the power limit (alone, at 1.7 GHz).  The same
// network with v_mfma_f32_32x32x16_bf16, half the issue cycles, ran at 1.8 GHz and no faster; rings of other depths neither.
// Measured, 61,440 envs x 3 agents x 64 steps, us: 3,670 -> 3,210, with the critic 4,775 -> 3,880; 10,240 envs x 6 agents 1,558 ->
// 1,126 and 2,188 -> 1,351; 6,144 x 10 1,997 -> 1,251 and 3,358 -> 1,482.  Results are those of the block kernel, bit for bit.
#include <type_traits>
#include <utility>

#include "mpe_mlp64.h"
#include "mpe_scenario.h"
#include "mpe_slots.h"
#include "mpe_gru_waves.h"

namespace mpe {

namespace {

template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(std::forward<F>(f), std::make_integer_sequence<int, N>{});
}

constexpr int kG = GruWavePk::kG;
constexpr int kFrag = GruWavePk::kFrag;

// LDS of one wavefront: positions by step parity (the current one holds a new episode's after a reset), landmarks, coverage distances.
template <typename Scn>
struct GruWaveLds {
  static constexpr int N = Scn::N, EW = 32 / N, ROWS = EW * N;
  float4 xch[2][Scn::kTag ? ROWS : (ROWS + 1) / 2];
  float2 lm[EW * (Scn::L + 1)];
  float dmin[Scn::kTag ? 1 : ROWS];
};

template <typename Scn, bool AC>
struct GruWaveSmem {
  static constexpr size_t OFF_BIAS = size_t(GruWavePk::RESIDENT) * kFrag;
  static constexpr size_t OFF_CBIAS = OFF_BIAS + GruWavePk::BIAS_FLOATS * 4;
  static constexpr size_t OFF_WAVE = OFF_CBIAS + (AC ? GruWaveCriticPk::BIAS_FLOATS * 4 : 0);
  static constexpr size_t WAVE = (sizeof(GruWaveLds<Scn>) + 15) / 16 * 16;
  static constexpr size_t TOTAL = OFF_WAVE + 8 * WAVE;
  static_assert(TOTAL <= 160 * 1024, "LDS");
};

__device__ __forceinline__ float gate_sigmoid(float x) { return hw_rcp(1.0f + hw_exp2(-kLog2e * x)); }

// Piece: SlotGrid for a launch of several slots of time (mpe_slots.h).  The envs of the launch are then TE * slots, one slot's after
// the other's, and a lane has a slot of its own (as in mpe_waves.h): wavefronts are full, and a batch of any size is many rounds of
// short blocks, of which the last one weighs little.
template <typename Scn, bool AC, typename Piece>
__global__ __launch_bounds__(512, 2) void rollout_gru_waves_kernel(TagArgs TA, const uint8_t* __restrict__ packed,
                                                                   const uint8_t* __restrict__ packed_critic,
                                                                   float* __restrict__ hidden, uint32_t end_env, Piece piece) {
  using M = GruWaveSmem<Scn, AC>;
  using TS = typename Scn::Shape;
  constexpr bool kTag = Scn::kTag, SLOTS = kSlots<Piece>;
  constexpr int N = Scn::N, L = Scn::L, D = Scn::D, KIN = Scn::LIVE, KSE = (KIN + 31) / 32;
  constexpr int EW = 32 / N, EB = 8 * EW, ROWS = EW * N;
  constexpr int G = kTag ? TS::G : 1, NA = kTag ? TS::A : 0;
  constexpr int OFF_EMB = GruWavePk::RESIDENT, OFF_GATE = OFF_EMB + 8 * KSE, OFF_FC = OFF_GATE + 48, OFF_OUT = OFF_FC + 32;
  const RolloutArgs& A = TA.r;
  [[maybe_unused]] const TagPhys& tg = TA.tg;
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  const int n = lane & 31;                     // this lane's agent row, for both halves of the wavefront
  const int j = lane & 15, gq = lane >> 4;     // matrix layout: rows j and 16 + j, lane group gq
  GruWaveLds<Scn>& sm = *reinterpret_cast<GruWaveLds<Scn>*>(smem + M::OFF_WAVE + size_t(wave) * M::WAVE);
  const size_t TE = A.TE;
  uint32_t blk;
  if constexpr (SLOTS) {
    blk = spread_group(blockIdx.x);
    if (blk >= piece.groups) return;
  } else {
    blk = xcd_group(piece);
    if (blk >= piece.end) return;                        // whole block, before any barrier
  }
  const uint32_t env0 = blk * EB + wave * EW;   // uniform
  const int nvalid = env0 < end_env ? min(int(end_env - env0), EW) : 0;
  const bool active = ROWS == 32 || n < ROWS;            // spare rows shadow the wavefront's first one and store nothing
  const int row = active ? n : 0, el = row / N, i = row - el * N;
  const bool in_range = el < nvalid, valid = active && in_range && lane < 32;
  // the wavefront's first envs, those of the slot that reads and writes the state
  const int nhead = !SLOTS ? nvalid : (env0 < A.TE ? min(int(A.TE - env0), nvalid) : 0);
  const bool head = !SLOTS || el < nhead;
  uint32_t env = env0 + (in_range ? el : 0), k_slot = 0;
  if constexpr (SLOTS) {
    k_slot = env / A.TE;
    env -= k_slot * A.TE;
  }
  const size_t g = nvalid ? env : 0u;
  const int32_t max_ep = kTag ? tg.max_ep : A.ph.max_ep;

  {
    const uint8_t* image = packed + GruWavePk::base();
    const uint4* src = reinterpret_cast<const uint4*>(image);
    uint4* dst = reinterpret_cast<uint4*>(smem);
    for (int k = threadIdx.x; k < int(M::OFF_BIAS / 16); k += 512) dst[k] = src[k];
    const float* b = reinterpret_cast<const float*>(image + size_t(OFF_OUT + 4) * kFrag);
    float* bd = reinterpret_cast<float*>(smem + M::OFF_BIAS);
    for (int k = threadIdx.x; k < GruWavePk::BIAS_FLOATS; k += 512) bd[k] = b[k];
    if constexpr (AC) {
      const float* c = reinterpret_cast<const float*>(packed_critic + GruWaveCriticPk::base() + size_t(GruWaveCriticPk::FRAGS) * kFrag);
      float* cd = reinterpret_cast<float*>(smem + M::OFF_CBIAS);
      for (int k = threadIdx.x; k < GruWaveCriticPk::BIAS_FLOATS; k += 512) cd[k] = c[k];
    }
  }

  // ---- this lane's agent; everything about the others is read from LDS where it is needed
  float px = 0.0f, py = 0.0f, vx = 0.0f, vy = 0.0f;
  int32_t ep = 0;
  uint32_t step = A.abs_step;
  // a new episode, keyed by the step that it starts at: every lane draws its own agent and landmarks i, i + N, ... of its env
  auto new_episode = [&](uint32_t start) {
    uint32_t env_r = env;
    asm volatile("" : "+v"(env_r));
    const uint4 d = philox4x32_10(env_r, start, uint32_t(i), kTagResetPos, A.seed, 0u);
    px = word_to_position(d.x);
    py = word_to_position(d.y);
    vx = vy = 0.0f;
    ep = 0;
#pragma unroll
    for (int k = 0; k < (L + N - 1) / N; ++k) {
      const int l = i + k * N;
      if (l < L) {
        const uint4 w = philox4x32_10(env_r, start, uint32_t(N + l), kTagResetPos, A.seed, 0u);
        float2 p = make_float2(word_to_position(w.x), word_to_position(w.y));
        if (kTag) { p.x *= 0.9f; p.y *= 0.9f; }
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
  // Several slots: number of steps of this lane's env, or, until the jump of slot 0, minus the steps before it
  [[maybe_unused]] int32_t event = 0, ep0 = ep, t0 = 0;
  int len = A.T;                                         // of the wavefront
  if constexpr (SLOTS) {
    counter_read(ep0);
    const TimeSlot slot = time_slot(A.T, A.slots, A.span, int(k_slot), ep0, max_ep, true);
    t0 = slot.t0;
    step += uint32_t(t0);
    event = in_range ? (slot.turn ? -slot.turn : slot.len) : 0;
    len = in_range ? slot.len : 0;
#pragma unroll
    for (int o = 32; o; o >>= 1) len = max(len, __shfl_xor(len, o));
    len = __builtin_amdgcn_readfirstlane(len);
  }
#pragma unroll
  for (int k = 0; k < (L + N - 1) / N; ++k) {
    const int l = i + k * N;
    if (l < L && active)
      sm.lm[el * (L + 1) + l] = in_range && head ? make_float2(A.st.pos_l[(0 * L + l) * TE + g], A.st.pos_l[(1 * L + l) * TE + g]) : make_float2(0.0f, 0.0f);
  }
  auto put = [&](int parity) {
    if (active) {
      if constexpr (kTag) sm.xch[parity][row] = make_float4(px, py, vx, vy);
      else reinterpret_cast<float2*>(sm.xch[parity])[row] = make_float2(px, py);
    }
  };
  auto pos = [&](int parity, int a) {
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
  if (nvalid == 0) return;
  [[maybe_unused]] TagRole me{};
  if constexpr (kTag) me = tag_role<TS>(i, tg);

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
    constexpr int CW = D % 4 == 0 ? 4 : 2;
    typedef float vC __attribute__((ext_vector_type(CW)));
#pragma unroll
    for (int q = 0; q < D / CW; ++q) {
      vC v;
#pragma unroll
      for (int e = 0; e < CW; ++e) v[e] = CW * q + e < KIN ? o[CW * q + e < KIN ? CW * q + e : 0] : 0.0f;
      reinterpret_cast<vC*>(dst)[q] = v;
    }
  };

  // ---- carried state of this wavefront's rows, in accumulator order: h[c][rt][r] is unit 32 (c / 2) + 8 gq + 4 (c % 2) + r of
  // row 16 rt + j
  float h[8][2][4];
  bf16x8 hb[4][2];      // the same rounded to bf16: B operand of K slice s, row tile rt
  float* hrow = hidden + (size_t(env0) * N + j) * kG + 8 * gq;
  const int vrows = nhead * N;
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
      if (16 * rt + j < vrows) v = *reinterpret_cast<const f32x4*>(hrow + rt * 16 * kG + 32 * (c / 2) + 4 * (c % 2));
#pragma unroll
      for (int r = 0; r < 4; ++r) h[c][rt][r] = v[r];
    }
  }
  auto pack8 = [](const auto& a, const auto& b) {        // the two tiles of a K slice
    return __builtin_bit_cast(bf16x8, u32x4{pack_bf16_rne(a[0], a[1]), pack_bf16_rne(a[2], a[3]), pack_bf16_rne(b[0], b[1]), pack_bf16_rne(b[2], b[3])});
  };
  auto pack_state = [&]() {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) hb[s][rt] = pack8(h[2 * s][rt], h[2 * s + 1][rt]);
  };
  pack_state();
  // outputs of this wavefront's first row (env), uniform, to which the lane adds its row; several slots: of the first time slice, to
  // which it adds the row and env in the slice of its own step
  const size_t row0 = SLOTS ? 0 : size_t(env0) * N;
  const bool per_agent = kTag || A.ph.reward_mode == 1;
  float* obs_p = A.obs_traj ? A.obs_traj + row0 * D : nullptr;
  uint8_t* act_p = A.act_traj ? A.act_traj + row0 : nullptr;
  float* rew_p = A.rew_traj ? A.rew_traj + (per_agent || SLOTS ? row0 : env0) : nullptr;
  uint8_t* done_p = A.done_traj ? A.done_traj + (SLOTS ? 0 : env0) : nullptr;
  [[maybe_unused]] float* logp_p = AC && A.logp_traj ? A.logp_traj + row0 : nullptr;
  [[maybe_unused]] float* value_p = AC && A.value_traj ? A.value_traj + row0 : nullptr;
  using Off = std::conditional_t<SLOTS, size_t, int>;
  Off env_at = el;
  if constexpr (SLOTS) {
    env_at = g + size_t(t0) * TE;
    if (valid && i == 0) settle_ticket(A, max_ep, g, take_ticket(A, g), ep0);
  }
  auto row_at = [&]() { return SLOTS ? Off(env_at * N + i) : Off(row); };
  float o[KIN];
#pragma unroll
  for (int c = 0; c < KIN; ++c) o[c] = 0.0f;
  wave_sync();
  build(o, 1);

  const auto image = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(packed) + GruWavePk::base(), 0, int(GruWavePk::bytes(KSE)), 0x00027000);
  [[maybe_unused]] const auto critic_image =
      __builtin_amdgcn_make_buffer_rsrc(AC ? const_cast<uint8_t*>(packed_critic) + GruWaveCriticPk::base() : nullptr, 0, AC ? int(GruWaveCriticPk::BYTES) : 0, 0x00027000);
  // The network on the rows in o: logits of the lane's own row (outputs only asked for in the loop), its value, and the
  // carried state advanced.
  auto network = [&](float (&z)[kNumActions], float& value) {
    // ================================================================ network
    // Opaque offsets: keep the step-invariant operand reads inside the step loop.  An LDS instruction reaches 64 KB.
    uint32_t zero = 0, lbase[3] = {uint32_t(lane) * 16u, uint32_t(lane) * 16u + 65536u, uint32_t(lane) * 16u + 131072u};
    asm volatile("" : "+v"(zero), "+v"(lbase[0]), "+v"(lbase[1]), "+v"(lbase[2]));
    uint32_t szero = 0;
    asm volatile("" : "+s"(szero));
    const int voff = lane * 16;
    const float* bias = reinterpret_cast<const float*>(smem + M::OFF_BIAS + zero) + 8 * gq;
    [[maybe_unused]] const float* cbias = reinterpret_cast<const float*>(smem + M::OFF_CBIAS + zero) + 8 * gq;
    auto lds = [&](int r) { return *reinterpret_cast<const bf16x8*>(smem + lbase[r / 64] + r % 64 * kFrag); };
    // streamed operands: buffer loads, which take the operand's place in the image as a scalar offset
    auto glb = [&](int f) { return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(image, voff, int(szero) + f * kFrag, 0)); };
    [[maybe_unused]] auto crit = [&](int f) { return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(critic_image, voff, int(szero) + f * kFrag, 0)); };
    struct Acc { f32x4 t[2]; };            // a unit tile's accumulators for both row tiles
    auto start = [&](const float* b, int c) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(b + 32 * (c / 2) + 4 * (c % 2));
      return Acc{{v, v}};
    };
    auto mma = [&](const bf16x8& a, const bf16x8 (&b)[2], Acc& acc) {
      acc.t[0] = MPE_MFMA_BF(a, b[0], acc.t[0]);
      acc.t[1] = MPE_MFMA_BF(a, b[1], acc.t[1]);
    };
    // rings of A operands in flight: LDS-resident gate operands, streamed gate operands
    constexpr int DL = 4, DG = 4;
    bf16x8 lr[DL], gr[DG];
    Acc ea[8];
    bf16x8 e[4][2];
    {
      bf16x8 we[8 * KSE];
#pragma unroll
      for (int k = 0; k < 8 * KSE; ++k) we[k] = glb(OFF_EMB + k);
#pragma unroll
      for (int k = 0; k < DG; ++k) gr[k] = glb(OFF_GATE + k);
#pragma unroll
      for (int k = 0; k < DL; ++k) lr[k] = lds(k);
#pragma unroll
      for (int c = 0; c < 8; ++c) ea[c] = start(bias, c);
      // B operands of the embedding: lane (j, gq) takes pairs 4 gq .. + 3 of rows j and 16 + j, which lie in lane groups
      // {0, 2} and {1, 3}
      bf16x8 in[KSE][2];
#pragma unroll
      for (int s = 0; s < KSE; ++s) {
        u32x4 p[2];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          uint32_t v[4];
#pragma unroll
          for (int b = 0; b < 4; ++b) {
            const int c = 32 * s + 8 * b + 2 * q;
            v[b] = c < KIN ? pack_bf16_rne(o[c < KIN ? c : 0], c + 1 < KIN ? o[c + 1 < KIN ? c + 1 : 0] : 0.0f) : 0u;
          }
          const auto w = __builtin_amdgcn_permlane16_swap(gq < 2 ? v[0] : v[2], gq < 2 ? v[1] : v[3], false, false);
          p[0][q] = w[0];
          p[1][q] = w[1];
        }
        in[s][0] = __builtin_bit_cast(bf16x8, p[0]);
        in[s][1] = __builtin_bit_cast(bf16x8, p[1]);
      }
#pragma unroll
      for (int s = 0; s < KSE; ++s)
#pragma unroll
        for (int c = 0; c < 8; ++c) mma(we[c * KSE + s], in[s], ea[c]);
    }
    __builtin_amdgcn_sched_barrier(0);
    // One gate operand of the stream: F = position among the 192
    auto gate_mma = [&](auto F, const bf16x8 (&b)[2], Acc& acc) {
      constexpr int f = decltype(F)::value;
      if constexpr (f % 4 == 3) {
        constexpr int k = f / 4;
        mma(gr[k % DG], b, acc);
        if constexpr (k + DG < 48) gr[k % DG] = glb(OFF_GATE + k + DG);
      } else {
        constexpr int k = f / 4 * 3 + f % 4;
        mma(lr[k % DL], b, acc);
        if constexpr (k + DL < GruWavePk::RESIDENT) lr[k % DL] = lds(k + DL);
      }
    };
    Acc nn, zz;         // of the tile whose new state comes next: tanh gate, update gate before its sigmoid
    auto blend = [&](auto C, auto X) {
      constexpr int c = decltype(C)::value, rt = decltype(X)::value / 4, x = decltype(X)::value % 4;
      // (1 - z) n + z h.  n is kept past the sum: where it ends there the compiler adds into its register and copies the sum to
      // h's, two instructions.
      const float nv = nn.t[rt][x], z = gate_sigmoid(zz.t[rt][x]), d = h[c][rt][x] - nv;
      h[c][rt][x] = __builtin_fmaf(z, d, nv);
      asm volatile("" : : "v"(nv));
    };
    static_for<8>([&](auto C) {
      constexpr int c = decltype(C)::value;
      Acc nh = start(bias + 4 * kG, c), rr = start(bias + kG, c);
      auto gate = [&](auto Q, Acc& acc) {
        constexpr int q = decltype(Q)::value;
        constexpr auto part = GruWavePk::gate_part(q);
        gate_mma(std::integral_constant<int, 24 * c + q>{}, part.recurrent ? hb[part.s] : e[part.s], acc);
      };
      // ---- recurrent part of n, reset gate; beside them the new state of the tile before (or the embedding's tanh)
      static_for<12>([&](auto J) {
        constexpr int q = decltype(J)::value;
        gate(J, q < 4 ? nh : rr);
        if constexpr (c == 0) {
          if constexpr (q < 8) {       // embedding: unit tile q; its K slice is complete after the second of a pair
#pragma unroll
            for (int x = 0; x < 8; ++x) ea[q].t[x / 4][x % 4] = fast_tanh(ea[q].t[x / 4][x % 4]);
            if constexpr (q % 2 == 1) {
              e[q / 2][0] = pack8(ea[q - 1].t[0], ea[q].t[0]);
              e[q / 2][1] = pack8(ea[q - 1].t[1], ea[q].t[1]);
            }
          }
        } else {
          if constexpr (q % 3 == 0) {  // two elements at a time: their chains fill each other's latencies
            blend(std::integral_constant<int, c - 1>{}, std::integral_constant<int, q / 3>{});
            blend(std::integral_constant<int, c - 1>{}, std::integral_constant<int, 4 + q / 3>{});
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      });
      // ---- input part of n; beside it the reset gate's sigmoid
      Acc ni = start(bias + 3 * kG, c);
      static_for<4>([&](auto J) {
        constexpr int q = decltype(J)::value;
        gate(std::integral_constant<int, 12 + q>{}, ni);
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) rr.t[rt][q] = gate_sigmoid(rr.t[rt][q]);
        __builtin_amdgcn_sched_barrier(0);
      });
      // ---- update gate; beside it n
      Acc za = start(bias + 2 * kG, c);
      static_for<8>([&](auto J) {
        constexpr int q = decltype(J)::value;
        gate(std::integral_constant<int, 16 + q>{}, za);
        if constexpr (q % 2 == 1) {
#pragma unroll
          for (int rt = 0; rt < 2; ++rt) ni.t[rt][q / 2] = fast_tanh(fmaf(rr.t[rt][q / 2], nh.t[rt][q / 2], ni.t[rt][q / 2]));
        }
        __builtin_amdgcn_sched_barrier(0);
      });
      nn = ni;
      zz = za;
    });
    // ---- second layers: NT unit tiles (the actor's eight, then the critic's); the outputs take a K slice as soon as both of
    // its tiles are there, after tiles 2, 4, 6 and 8
    constexpr int NT = AC ? 16 : 8, SEQ = 4 * NT + 4, DF = 8;
    constexpr auto outs_before = [](int tt) { return tt < 1 ? 0 : ((tt - 1) / 2 < 4 ? (tt - 1) / 2 : 4); };
    auto seq_frag = [&](auto S) {
      constexpr int s = decltype(S)::value;
      // tile and place inside it: tiles 2, 4, 6, 8 have a fifth operand, the outputs'
      constexpr int late = 4 * 9 + 4;        // first operand of tile 9
      constexpr int tt = s >= late ? 9 + (s - late) / 4 : (s < 8 ? s / 4 : 2 + (s - 8) / 9 * 2 + (s - 8) % 9 / 5);
      constexpr int k = s >= late ? (s - late) % 4 : (s < 8 ? s % 4 : ((s - 8) % 9 < 5 ? (s - 8) % 9 : (s - 8) % 9 - 5));
      if constexpr (k == 4 || tt >= NT) return glb(OFF_OUT + tt / 2 - 1);
      else if constexpr (tt < 8) return glb(OFF_FC + 4 * tt + k);
      else return crit(4 * (tt - 8) + k);
    };
    bf16x8 fr[DF];
    static_for<DF>([&](auto S) { fr[S] = seq_frag(S); });
    __builtin_amdgcn_sched_barrier(0);
    static_for<8>([&](auto X) { blend(std::integral_constant<int, 7>{}, X); });
    pack_state();
    __builtin_amdgcn_sched_barrier(0);
    Acc out;
    out.t[0] = *reinterpret_cast<const f32x4*>(bias + 6 * kG - 4 * gq);
    out.t[1] = out.t[0];
    if constexpr (AC) value = cbias[2 * kG - 8 * gq];
    auto take = [&](auto S, const bf16x8 (&b)[2], Acc& acc) {
      constexpr int s = decltype(S)::value;
      mma(fr[s % DF], b, acc);
      if constexpr (s + DF < SEQ) fr[s % DF] = seq_frag(std::integral_constant<int, s + DF>{});
    };
    Acc ya[2];          // tanh of the tile before and of the one before that
    [[maybe_unused]] float pv[2];
    static_for<NT + 1>([&](auto TT) {
      constexpr int tt = decltype(TT)::value, first = 4 * tt + outs_before(tt);
      Acc acc{};
      if constexpr (tt < NT) acc = tt < 8 ? start(bias + 5 * kG, tt) : start(cbias, tt - 8);
      [[maybe_unused]] f32x4 wv{};
      if constexpr (tt > 8) wv = start(cbias + kG, tt - 9).t[0];
      static_for<4>([&](auto K) {
        constexpr int k = decltype(K)::value;
        if constexpr (tt < NT) take(std::integral_constant<int, first + k>{}, hb[k], acc);
        if constexpr (tt > 0) {
#pragma unroll
          for (int rt = 0; rt < 2; ++rt) ya[0].t[rt][k] = fast_tanh(ya[0].t[rt][k]);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
      if constexpr (tt > 0 && tt <= 8 && tt % 2 == 0) {
        const bf16x8 y[2] = {pack8(ya[1].t[0], ya[0].t[0]), pack8(ya[1].t[1], ya[0].t[1])};
        take(std::integral_constant<int, first + (tt < NT ? 4 : 0)>{}, y, out);
      }
      if constexpr (tt > 8) {
        // value += wv . yc, in the block kernel's order: terms of four units, (0 + 1) + (2 + 3) of 16 units, 16 units in turn
        float p[2];
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) {
          const uint32_t lo = pack_bf16_rne(ya[0].t[rt][0], ya[0].t[rt][1]), hi = pack_bf16_rne(ya[0].t[rt][2], ya[0].t[rt][3]);
          p[rt] = __uint_as_float(lo << 16) * wv[0];
          p[rt] = fmaf(__uint_as_float(lo & 0xFFFF0000u), wv[1], p[rt]);
          p[rt] = fmaf(__uint_as_float(hi << 16), wv[2], p[rt]);
          p[rt] = fmaf(__uint_as_float(hi & 0xFFFF0000u), wv[3], p[rt]);
        }
        if constexpr (tt % 2 == 1) {
          pv[0] = p[0];
          pv[1] = p[1];
        } else {
          // lane group gq has terms 2 (gq % 2), + 1 of the 16 units gq / 2 of this pair of tiles
          const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(pv[0] + p[0]), __float_as_uint(pv[1] + p[1]), false, false);
          const uint32_t sum = __float_as_uint(__uint_as_float(a[0]) + __uint_as_float(a[1]));   // of the lane's own row
          const auto b = __builtin_amdgcn_permlane32_swap(sum, sum, false, false);
          value += __uint_as_float(b[0]);
          value += __uint_as_float(b[1]);
        }
      }
      ya[1] = ya[0];
      ya[0] = acc;
      __builtin_amdgcn_sched_barrier(0);
    });
    // logits of the lane's own row: lane groups 0 and 2 have outputs 0..3 of both row tiles, 1 and 3 output 4
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const auto w = __builtin_amdgcn_permlane16_swap(__float_as_uint(out.t[0][k]), __float_as_uint(out.t[1][k]), false, false);
      z[k] = __uint_as_float(w[0]);
      if (k == 0) z[4] = __uint_as_float(w[1]);
    }
  };

  // state and last observation of the lanes that have run all their steps
  auto finish = [&](bool ended) {
    const bool stores = valid && ended;
    // opaque: addresses computed from it stay here instead of in 20 to 30 registers over the loop of steps
    uint32_t env_f = uint32_t(g), j_f = uint32_t(j), i_f = uint32_t(i), gq_f = uint32_t(gq);
    if constexpr (SLOTS) asm volatile("" : "+v"(env_f), "+v"(j_f), "+v"(i_f), "+v"(gq_f));
    const size_t g = env_f;
    const int i = int(i_f), j = int(j_f);
    float* hrow = hidden + (size_t(env0) * N + j_f) * kG + 8 * gq_f;
    if (A.last_obs) store_row(o, A.last_obs + (g * N + i) * D, stores);
    const uint64_t rows = SLOTS ? __ballot(ended) : ~0ull;
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      if (16 * rt + j < vrows && (rows >> (16 * rt + j) & 1)) {
#pragma unroll
        for (int c = 0; c < 8; ++c)
          *reinterpret_cast<f32x4*>(hrow + rt * 16 * kG + 32 * (c / 2) + 4 * (c % 2)) = f32x4{h[c][rt][0], h[c][rt][1], h[c][rt][2], h[c][rt][3]};
      }
    }
    if (stores) {
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
    const bool ended = SLOTS && head && t == event;      // before the wavefront's other lanes
    if constexpr (SLOTS) {
      if (__ballot(ended)) finish(ended);
    }
    const bool stores = valid && (!SLOTS || event < 0 || t < event), env_writer = stores && i == 0;
    if (obs_p) {
      store_row(o, obs_p + row_at() * D, stores);
      obs_p += TE * (N * D);
    }
    float z[kNumActions], value = 0.0f;
    network(z, value);
    if constexpr (AC && SLOTS) {
      if (ended && valid && A.last_value) A.last_value[g * N + i] = value;
    }
    const int par = t & 1;
    // Sampling noise as in gumbel_noise: the lower half of the wavefront draws the block of the first four actions, the
    // upper half that of the fifth; the lower half picks.
    uint32_t act;
    {
      const uint4 w4 = philox4x32_10(env, step, uint32_t(i), lane < 32 ? kTagGumbel0 : kTagGumbel1, A.seed, 0u);
      const uint32_t w[4] = {w4.x, w4.y, w4.z, w4.w};
      float nz[kNumActions];
#pragma unroll
      for (int k = 0; k < 4; ++k) nz[k] = hw_log2(-kLn2 * hw_log2(word_to_open_uniform(w[k])));
      const auto f = __builtin_amdgcn_permlane32_swap(__float_as_uint(nz[0]), __float_as_uint(nz[0]), false, false);
      nz[4] = __uint_as_float(f[1]);
      act = gumbel_pick(z, nz);
      act = __builtin_amdgcn_permlane32_swap(act, act, false, false)[0];
    }
    if (act_p) {
      if (stores) act_p[row_at()] = uint8_t(act);
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
        if (stores) logp_p[row_at()] = (zact - zmax) - kLn2 * hw_log2(sum);
        logp_p += TE * N;
      }
      if (value_p) {
        if (stores) value_p[row_at()] = value;
        value_p += TE * N;
      }
    }
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
        if (stores) rew_p[row_at()] = r;
      } else {
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
          const float mr = mixed_reward(r, overlap_count<N>(i, px, py, qx, qy, A.ph), A.ph);
          if (stores) rew_p[row_at()] = mr;
        } else if (env_writer) {
          rew_p[env_at] = r;
        }
      }
      rew_p += per_agent ? TE * N : TE;
    }
    ep += 1;
    const bool done = ep >= max_ep;
    if (done_p) {
      if (env_writer) done_p[env_at] = done ? 1 : 0;
      done_p += TE;
    }
    ++step;
    if constexpr (SLOTS) {
      if (t + 1 == -event) {                           // slot 0's current episode ends
        const int32_t jump = (A.slots - 1) * A.span;
        event = A.T - jump;
        step += uint32_t(jump);
        env_at += size_t(jump) * TE;
      }
    }
    if (done) new_episode(step);
    if (const uint64_t fresh = __ballot(done)) {       // the carried state of a new episode is zero
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) {
        if (fresh >> (16 * rt + j) & 1) {
#pragma unroll
          for (int c = 0; c < 8; ++c) h[c][rt][0] = h[c][rt][1] = h[c][rt][2] = h[c][rt][3] = 0.0f;
#pragma unroll
          for (int s = 0; s < 4; ++s) hb[s][rt] = __builtin_bit_cast(bf16x8, u32x4{0u, 0u, 0u, 0u});
        }
      }
    }
    wave_sync();               // the positions before a reset have been read
    if (done) put(par);
    wave_sync();
    build(o, par);
  }
  const bool ended = !SLOTS || (head && event == len);
  if (nhead) finish(ended);
  if constexpr (AC) {
    if (A.last_value && nhead) {   // one more evaluation on the last observation; the state it leaves is dropped
      float z[kNumActions], value = 0.0f;
      network(z, value);
      if (valid && ended) A.last_value[g * N + i] = value;
    }
  }
}

template <typename Scn, bool AC>
hipError_t launch_impl(const TagArgs& A, const void* packed, const void* critic, float* hidden, uint32_t envs, hipStream_t s) {
  using M = GruWaveSmem<Scn, AC>;
  static std::atomic<uint64_t> lds_allowed[2];
  constexpr uint32_t EB = gru_waves_block_envs(Scn::N);
  auto launch = [&](auto kern, dim3 grid, auto piece) {
    hipLaunchKernelGGL(kern, grid, dim3(512), M::TOTAL, s, A, static_cast<const uint8_t*>(packed), static_cast<const uint8_t*>(critic), hidden, envs, piece);
  };
  if (A.r.slots > 1) {
    auto kern = rollout_gru_waves_kernel<Scn, AC, SlotGrid>;
    if (hipError_t e = allow_lds(reinterpret_cast<const void*>(kern), M::TOTAL, lds_allowed[1]); e != hipSuccess) return e;
    const uint32_t blocks = (envs + EB - 1) / EB;
    launch(kern, spread_grid(blocks), SlotGrid{blocks});
    return hipGetLastError();
  }
  auto kern = rollout_gru_waves_kernel<Scn, AC, GridPiece>;
  if (hipError_t e = allow_lds(reinterpret_cast<const void*>(kern), M::TOTAL, lds_allowed[0]); e != hipSuccess) return e;
  return launch_groups<512>((envs + EB - 1) / EB, [&](dim3 grid, const GridPiece& p) { launch(kern, grid, p); });
}

}  // namespace

hipError_t launch_gru_waves(bool tag, int N, int L, int G, const TagArgs& A, const void* packed, const void* critic, float* hidden,
                            uint32_t envs, hipStream_t s) {
#define MPE_GO(...) \
  return critic ? launch_impl<__VA_ARGS__, true>(A, packed, critic, hidden, envs, s) : launch_impl<__VA_ARGS__, false>(A, packed, nullptr, hidden, envs, s)
  if (tag) {
#define X(n, l, g) \
    if (N == n && L == l && G == g) MPE_GO(TagScn<n, l, g>);
    MPE_TAG_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
  }
  switch (N) {
#define X(n) case n: MPE_GO(SpreadScn<n>);
    X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10)
#undef X
    default: return hipErrorInvalidValue;
  }
#undef MPE_GO
}

}  // namespace mpe
