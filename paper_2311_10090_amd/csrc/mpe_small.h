// Fused rollout for batches that leave the chip's SIMDs short of wavefronts: few environments, or many small
// training runs (the paper's IPPO setting is 16 environments per run, App. G).  Same networks (two tanh layers of
// width 64; Sec. 3.2, App. G), same arithmetic in the same order and therefore the same results, bit for bit, as
// the kernels for full batches in mpe_policy_f32.hip and mpe_tag.hip.
//
// What bounds it: the latency of one step.  A lone wavefront of a SIMD issues one vector instruction every 5.3 to 8
// cycles, whatever its neighbours on other SIMDs do, so the time of a step is the number of instructions on the
// longest path through it.  The kernel therefore cuts that path instead of the total work:
//  * a POLICY wavefront owns ONE 16-row tile (the smallest matrix tile).  Its four lane groups are clones of the
//    tile's rows: every lane holds the state of agent row `lane & 15`, so the operands of layer 1 come from the
//    lane's own registers and the logits come back by lane-group swaps, without a trip through LDS.  The weights
//    are stationary in registers (REGW) while a block has a CU to itself, else in LDS;
//  * everything that the next step does not wait for is done by SERVICE wavefronts, one lane per row and one step
//    behind: trajectory stores, rewards, log-probabilities; and by them one step AHEAD: the sampling noise and the
//    positions of an episode that is about to start (both are functions of the counter-based generator alone);
//  * in the actor-critic rollout, CRITIC wavefronts (one per tile, or fewer that take several tiles in turn where a block
//    would have more than 16 wavefronts) evaluate the critic one step behind.
// All wavefronts of a block meet at one block barrier per step; everything they exchange is double-buffered by
// step parity.
#pragma once

#include "mpe_mlp64.h"
#include "mpe_scenario.h"
#include "mpe_slot_cost.h"

namespace mpe {

namespace {

template <int N_>
struct SmallSpread : SpreadScn<N_> {
  using Net = NetShape<6 * N_, 4 * N_ + 2>;
};
template <int N_, int L_, int G_>
struct SmallTag : TagScn<N_, L_, G_> {
  using Net = NetShape<TagScn<N_, L_, G_>::D, TagScn<N_, L_, G_>::D>;
};

// ------------------------------------------------------------------------------ network of one 16-row tile
// Operands of one network: in registers for the whole rollout (REGW), or read from its image in LDS where used.
template <typename S, bool BF, bool REGW>
struct TileNet {
  using P = PkT<BF, S::kWideIn, S::kSlices1>;
  static constexpr int KS1 = S::kSlices1;
  static constexpr int T1 = BF ? 1 : (S::kWideIn ? 3 : 2), T2 = BF ? 1 : 2, T3 = (BF || S::kRowTerms) ? 1 : 3;
  bf16x8 r1[REGW ? 4 * KS1 * T1 : 1], r2[REGW ? 8 * T2 : 1], r3[2 * T3];
  const uint8_t* image;        // !REGW: W1A, W2A in LDS
  const float* bias;           // in LDS
  int lane;

  // `global`: the packed image of the block's run; `lds`: where its W1A + W2A are staged (unless REGW)
  __device__ __forceinline__ void init(const uint8_t* __restrict__ global, const uint8_t* lds, const float* bias_lds, int lane_) {
    image = lds;
    bias = bias_lds;
    lane = lane_;
    const bf16x8* g = reinterpret_cast<const bf16x8*>(global) + lane;
    if constexpr (REGW) {
#pragma unroll
      for (int k = 0; k < 4 * KS1 * T1; ++k) r1[k] = g[P::OFF_W1A / 16 + k * 64];
#pragma unroll
      for (int k = 0; k < 8 * T2; ++k) r2[k] = g[P::OFF_W2A / 16 + k * 64];
    }
#pragma unroll
    for (int k = 0; k < 2 * T3; ++k) r3[k] = g[P::OFF_W3A / 16 + k * 64];
  }
  __device__ __forceinline__ bf16x8 w1(int k, uint32_t zero) const {
    if constexpr (REGW) return r1[k];
    else return reinterpret_cast<const bf16x8*>(image + P::OFF_W1A + zero)[k * 64 + lane];
  }
  __device__ __forceinline__ bf16x8 w2(int k, uint32_t zero) const {
    if constexpr (REGW) return r2[k];
    else return reinterpret_cast<const bf16x8*>(image + P::OFF_W2A + zero)[k * 64 + lane];
  }

  // v: this lane's 8 layer-1 inputs per K slice (see policy_core); returns the layer-3 accumulators.  The products
  // of an accumulator are in the order of policy_core / policy_pair_bf.
  __device__ __forceinline__ f32x4 forward(const float (&v)[KS1][8]) const {
    uint32_t zero = 0;            // opaque: keeps step-invariant LDS reads inside the step loop (see policy_core)
    asm volatile("" : "+v"(zero));
    const float* b = bias + zero + 4 * (lane >> 4);
    f32x4 acc[4], acc2[4];
    if constexpr (BF) {
      bf16x8 in[KS1];
#pragma unroll
      for (int s = 0; s < KS1; ++s) {
        u32x4 p;
#pragma unroll
        for (int q = 0; q < 4; ++q) p[q] = pack_bf16_rne(v[s][2 * q], v[s][2 * q + 1]);
        in[s] = __builtin_bit_cast(bf16x8, p);
      }
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        acc[m] = *reinterpret_cast<const f32x4*>(b + 16 * m);
        acc2[m] = *reinterpret_cast<const f32x4*>(b + kH + 16 * m);
      }
#pragma unroll
      for (int s = 0; s < KS1; ++s)
#pragma unroll
        for (int m = 0; m < 4; ++m) acc[m] = MPE_MFMA_BF(w1(m * KS1 + s, zero), in[s], acc[m]);
      f32x4 z = *reinterpret_cast<const f32x4*>(b + 2 * kH);
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const bf16x8 h = tanh_pack_bf(acc[2 * s], acc[2 * s + 1]);
#pragma unroll
        for (int m = 0; m < 4; ++m) acc2[m] = MPE_MFMA_BF(w2(m * 2 + s, zero), h, acc2[m]);
      }
#pragma unroll
      for (int s = 0; s < 2; ++s) z = MPE_MFMA_BF(r3[s], tanh_pack_bf(acc2[2 * s], acc2[2 * s + 1]), z);
      return z;
    } else {
      Terms in[KS1];
#pragma unroll
      for (int s = 0; s < KS1; ++s) in[s] = split_operand(v[s]);
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        acc[m] = *reinterpret_cast<const f32x4*>(b + 16 * m);
        acc2[m] = *reinterpret_cast<const f32x4*>(b + kH + 16 * m);
      }
      if constexpr (S::kWideIn) {
        // the six cross terms, smallest first, the four tiles in turn (see mma_split)
#pragma unroll
        for (int s = 0; s < KS1; ++s)
#pragma unroll
          for (int x = 0; x < 6; ++x)
#pragma unroll
            for (int m = 0; m < 4; ++m) {
              constexpr int ta[6] = {2, 0, 1, 1, 0, 0};          // l h m m h h of the weights
              const bf16x8 a = w1((m * KS1 + s) * 3 + ta[x], zero);
              const bf16x8 c = (x == 0 || x == 3 || x == 5) ? in[s].h : (x == 1 ? in[s].l : in[s].m);
              acc[m] = MPE_MFMA_SPLIT(a, c, acc[m]);
            }
      } else {
        const bf16x8 lh = lane < 32 ? in[0].l : in[0].h;
#pragma unroll
        for (int x = 0; x < 3; ++x)
#pragma unroll
          for (int m = 0; m < 4; ++m)
            acc[m] = MPE_MFMA_SPLIT(w1(m * 2 + (x == 0 ? 1 : 0), zero), x == 0 ? lh : (x == 1 ? in[0].m : in[0].h), acc[m]);
      }
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const Terms h = tanh_split(acc[2 * s], acc[2 * s + 1]);
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
          for (int m = 0; m < 4; ++m)
            acc2[m] = MPE_MFMA_SPLIT(w2((m * 2 + s) * 2 + (x < 2 ? 1 : 0), zero), (x == 0 || x == 2) ? h.m : h.h, acc2[m]);
      }
      f32x4 z = *reinterpret_cast<const f32x4*>(b + 2 * kH);
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const Terms y = tanh_split(acc2[2 * s], acc2[2 * s + 1]);
        if constexpr (S::kRowTerms) {
          z = MPE_MFMA_SPLIT(r3[s], y.m, z);
          z = MPE_MFMA_SPLIT(r3[s], y.h, z);
        } else {
          Terms a;
          a.h = r3[s * 3];
          a.m = r3[s * 3 + 1];
          a.l = r3[s * 3 + 2];
          z = mma_split_act(a, y, z);
        }
      }
      return z;
    }
  }
};

// Value of lane group g of x in every lane group: out[g] (g = 0..3).
__device__ __forceinline__ void gather_groups(float x, float (&out)[4]) {
  const uint32_t u = __float_as_uint(x);
  const auto s = __builtin_amdgcn_permlane32_swap(u, u, false, false);        // [g0 g1 g0 g1], [g2 g3 g2 g3]
  const auto a = __builtin_amdgcn_permlane16_swap(s[0], s[0], false, false);  // g0 everywhere, g1 everywhere
  const auto b = __builtin_amdgcn_permlane16_swap(s[1], s[1], false, false);
  out[0] = __uint_as_float(a[0]);
  out[1] = __uint_as_float(a[1]);
  out[2] = __uint_as_float(b[0]);
  out[3] = __uint_as_float(b[1]);
}

// The five logits of row lane & 15 in every lane, from the layer-3 accumulators of its tile.
template <typename S, bool BF>
__device__ __forceinline__ void tile_logits(const f32x4& a, float (&z)[kNumActions]) {
  float g[4];
  if constexpr (!BF && S::kRowTerms) {   // lane group g: the three terms of output g, and term g of output 4
    gather_groups((a[0] + a[1]) + a[2], g);
#pragma unroll
    for (int k = 0; k < 4; ++k) z[k] = g[k];
    gather_groups(a[3], g);
    z[4] = (g[0] + g[1]) + g[2];
  } else {                               // lane group 0: outputs 0..3; lane group 1: output 4
    gather_groups(a[0], g);
    z[0] = g[0];
    z[4] = g[1];
#pragma unroll
    for (int k = 1; k < 4; ++k) {
      gather_groups(a[k], g);
      z[k] = g[0];
    }
  }
}

// ------------------------------------------------------------------------------ LDS plan of a block
template <typename Scn, int EB, bool AC, bool BF, bool REGW>
struct SmallSmem {
  using Net = typename Scn::Net;
  using P = PkT<BF, Net::kWideIn, Net::kSlices1>;
  static constexpr int N = Scn::N, D = Scn::D, L = Scn::L, B = EB * N;
  static constexpr int TILES = B / 16, SERVICE = (B + 63) / 64;
  // critic wavefronts: one per tile where the block's 16 wavefronts allow it, else each takes several in turn
  static constexpr int CRITICS = !AC ? 0 : (2 * TILES + SERVICE <= 16 ? TILES : 16 - TILES - SERVICE);
  static constexpr int WAVES = TILES + CRITICS + SERVICE;
  static_assert(B % 16 == 0 && WAVES <= 16, "whole 16-row tiles");
  static constexpr size_t W = REGW ? 0 : P::LDS_BYTES;             // staged W1A + W2A of one network
  static constexpr size_t OFF_CRITIC = W;
  static constexpr size_t OFF_BIAS = W * (AC ? 2 : 1);
  static constexpr size_t OFF_CBIAS = OFF_BIAS + P::BIAS_BYTES;
  static constexpr size_t OFF_OBS = OFF_CBIAS + (AC ? P::BIAS_BYTES : 0);          // [2][B][D] floats (+ 64 bytes read past the end)
  static constexpr size_t OBS = size_t(B) * D * 4;
  static constexpr size_t OFF_XCH = OFF_OBS + 2 * OBS + 64;                         // [2][B] float4: new position (and velocity)
  static constexpr size_t OFF_NOISE = OFF_XCH + size_t(2) * B * 16;                 // [2][5][B]
  // AC: the logits of a step go to the service wavefront in the place of its noise, which has been read by then
  static constexpr size_t OFF_ACT = OFF_NOISE + size_t(2) * kNumActions * B * 4;    // [2][B]
  static constexpr int ENT = N + L;                                                 // entities of an env
  static constexpr size_t OFF_RESET = OFF_ACT + size_t(2) * B * 4;                  // [2][EB][N + L] float2
  static constexpr size_t TOTAL = OFF_RESET + size_t(2) * EB * ENT * 8;
  static_assert(OFF_OBS % 16 == 0 && OBS % 16 == 0 && OFF_XCH % 16 == 0 && OFF_RESET % 8 == 0 && TOTAL <= 160 * 1024, "LDS");
};

// MINW: wavefronts per SIMD the register budget is set for.
template <typename Scn, int EB, bool AC, bool BF, bool REGW, int MINW, typename Piece>
__global__ __launch_bounds__((SmallSmem<Scn, EB, AC, BF, REGW>::WAVES * 64), MINW) void rollout_small_kernel(
    TagArgs TA, const uint8_t* __restrict__ packed, const uint8_t* __restrict__ packed_critic, int per_run_weights, Piece piece) {
  using M = SmallSmem<Scn, EB, AC, BF, REGW>;
  using P = typename M::P;
  using S = typename Scn::Net;
  using TS = typename Scn::Shape;                      // predator-prey only
  constexpr bool kTag = Scn::kTag, SLOTS = kSlots<Piece>;
  constexpr int N = Scn::N, L = Scn::L, D = Scn::D, B = M::B, TILES = M::TILES, KS1 = S::kSlices1;
  constexpr int G = kTag ? TS::G : 1, NA = kTag ? TS::A : 0;
  const RolloutArgs& A = TA.r;
  [[maybe_unused]] const TagPhys& tg = TA.tg;
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  float* obs_tile = reinterpret_cast<float*>(smem + M::OFF_OBS);
  float4* xch = reinterpret_cast<float4*>(smem + M::OFF_XCH);
  float* noise = reinterpret_cast<float*>(smem + M::OFF_NOISE);
  [[maybe_unused]] float* logits = noise;
  uint32_t* acts = reinterpret_cast<uint32_t*>(smem + M::OFF_ACT);
  float2* fresh = reinterpret_cast<float2*>(smem + M::OFF_RESET);

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  const size_t TE = A.TE;
  int k_slot;
  uint32_t grp;
  if (!take_slot(A, piece, k_slot, grp)) return;                           // whole block, before any barrier
  const size_t g0 = size_t(grp) * EB;
  const int nvalid = TE - g0 < size_t(EB) ? int(TE - g0) : EB;
  const size_t run_off = per_run_weights ? size_t(uint32_t(g0) / A.E) * P::RUN_BYTES : 0;
  const int32_t max_ep = kTag ? tg.max_ep : A.ph.max_ep;
  const TimeSlot slot = group_slot<SLOTS>(A, k_slot, max_ep, g0, nvalid, lane);
  const bool head = k_slot == 0;                       // the slot that reads and writes the envs' state

  // ---- biases (and, unless the operands stay in registers, the staged weights)
  {
    constexpr int THREADS = M::WAVES * 64;
    auto stage = [&](const uint8_t* src, size_t w_off, size_t b_off) {
      const uint4* s4 = reinterpret_cast<const uint4*>(src);
      if constexpr (!REGW) {
        uint4* d4 = reinterpret_cast<uint4*>(smem + w_off);
        for (int k = threadIdx.x; k < int(P::LDS_BYTES / 16); k += THREADS) d4[k] = s4[k];
      }
      const uint4* sb = reinterpret_cast<const uint4*>(src + P::OFF_BIAS);
      uint4* db = reinterpret_cast<uint4*>(smem + b_off);
      for (int k = threadIdx.x; k < int(P::BIAS_BYTES / 16); k += THREADS) db[k] = sb[k];
    };
    stage(packed + run_off, 0, M::OFF_BIAS);
    if constexpr (AC) stage(packed_critic + run_off, M::OFF_CRITIC, M::OFF_CBIAS);
    // trailing zeros of the rows (and what layer 1 reads past the last one): never written again
    for (int k = threadIdx.x; k < int((2 * M::OBS + 64) / 16); k += THREADS) reinterpret_cast<uint4*>(obs_tile)[k] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
  }

  if (wave < TILES) {
    // ================================================================ policy wavefront: tile `wave`
    __builtin_amdgcn_s_setprio(2);
    const int j = lane & 15, gq = lane >> 4;
    const int row = wave * 16 + j, el = row / N, i = row - el * N;
    const size_t g = g0 + el;
    const bool valid = g < TE;
    TileNet<S, BF, REGW> net;
    net.init(packed + run_off, smem, reinterpret_cast<const float*>(smem + M::OFF_BIAS), lane);
    float px = 0.0f, py = 0.0f, vx = 0.0f, vy = 0.0f;
    float qx[N], qy[N], lx[L + 1], ly[L + 1];
    [[maybe_unused]] float gvx[G], gvy[G];
    int32_t ep = 0;
#pragma unroll
    for (int a = 0; a < N; ++a) qx[a] = qy[a] = 0.0f;
#pragma unroll
    for (int k = 0; k < L + 1; ++k) lx[k] = ly[k] = 0.0f;
#pragma unroll
    for (int k = 0; k < G; ++k) gvx[k] = gvy[k] = 0.0f;
    // a new episode's positions, drawn by the service wavefronts
    auto take_fresh = [&](int parity) {
      const float2* f = fresh + (size_t(parity) * EB + el) * M::ENT;
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
    } else if (valid) {
#pragma unroll
      for (int a = 0; a < N; ++a) {
        qx[a] = A.st.pos_a[(0 * N + a) * TE + g];
        qy[a] = A.st.pos_a[(1 * N + a) * TE + g];
      }
#pragma unroll
      for (int k = 0; k < L; ++k) {
        lx[k] = A.st.pos_l[(0 * L + k) * TE + g];
        ly[k] = A.st.pos_l[(1 * L + k) * TE + g];
      }
      if constexpr (kTag) {
#pragma unroll
        for (int k = 0; k < G; ++k) {
          gvx[k] = A.st.vel_a[(0 * N + NA + k) * TE + g];
          gvy[k] = A.st.vel_a[(1 * N + NA + k) * TE + g];
        }
      }
      vx = A.st.vel_a[(0 * N + i) * TE + g];
      vy = A.st.vel_a[(1 * N + i) * TE + g];
      ep = A.st.ep_step[g];
    }
#pragma unroll
    for (int a = 0; a < N; ++a) {
      if (a == i) { px = qx[a]; py = qy[a]; }
    }
    [[maybe_unused]] TagRole me{};
    if constexpr (kTag) me = tag_role<TS>(i, tg);

    // The row of the next step: into the LDS tile (for the stores and the critic), and this lane's inputs of layer 1.
    constexpr int OW = S::kWideIn ? 32 * KS1 : 16;                      // row entries that layer 1 reads, padded
    constexpr int LIVE = S::KIN;                                       // entries that are not always zero
    float in[KS1][8];
    auto next_obs = [&](int parity) {
      float o[OW];
#pragma unroll
      for (int c = 0; c < OW; ++c) o[c] = 0.0f;
      agent_obs<Scn>(o, i, px, py, vx, vy, qx, qy, lx, ly, gvx, gvy);
      float* rows = obs_tile + size_t(parity) * B * D;
      if (gq == 0) {
        float2* dst = reinterpret_cast<float2*>(rows + row * D);
#pragma unroll
        for (int c = 0; c < LIVE / 2; ++c) dst[c] = make_float2(o[2 * c], o[2 * c + 1]);
      }
      if constexpr (!S::kWideIn) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          float lo = o[e], hi = o[8 + e];
          asm("" : "+v"(lo), "+v"(hi));   // a select of registers, not of array addresses
          in[0][e] = (gq & 1) ? hi : lo;
        }
      } else {
        wave_sync();
#pragma unroll
        for (int s = 0; s < KS1; ++s) load_row_inputs<S>(rows + wave * 16 * D, j, gq, s, in[s]);
      }
    };
    next_obs(0);
    if (SLOTS) counter_read(ep);
    __syncthreads();   // first observations and the noise of step 0
    for (int t = 0; t < slot.len; ++t) {
      const int par = t & 1;
      float nz[kNumActions], z[kNumActions];
#pragma unroll
      for (int k = 0; k < kNumActions; ++k) nz[k] = noise[(par * kNumActions + k) * B + row];
      tile_logits<S, BF>(net.forward(in), z);
      uint32_t act = 0;
      float best = -INFINITY;
#pragma unroll
      for (int k = 0; k < kNumActions; ++k) {
        const float v = fmaf(-kLn2, nz[k], z[k]);
        if (v > best) { best = v; act = uint32_t(k); }
      }
      if constexpr (kTag) tag_move<TS>(act, i, me, tg, px, py, vx, vy, qx, qy, lx, ly);
      else agent_move<N>(act, i, A.ph, px, py, vx, vy, qx, qy);
      if (gq == 0) {
        xch[par * B + row] = make_float4(px, py, vx, vy);
        acts[par * B + row] = act;
        if constexpr (AC) {
#pragma unroll
          for (int k = 0; k < kNumActions; ++k) logits[(par * kNumActions + k) * B + row] = z[k];
        }
      }
      __syncthreads();
      ep += 1;
      const bool done = ep >= max_ep;
#pragma unroll
      for (int a = 0; a < N; ++a) {
        const float4 p = xch[par * B + el * N + a];
        qx[a] = p.x;
        qy[a] = p.y;
        if constexpr (kTag) {
          if (a >= NA) {
            gvx[a - NA] = p.z;
            gvy[a - NA] = p.w;
          }
        }
      }
      if (done) {
        take_fresh(par);
        if constexpr (kTag) {
#pragma unroll
          for (int k = 0; k < G; ++k) gvx[k] = gvy[k] = 0.0f;
        }
        vx = vy = 0.0f;
        ep = 0;
      }
      next_obs(par ^ 1);
    }
    __syncthreads();   // last observations
    if (valid && gq == 0 && head) {
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
  } else if (AC && wave < TILES + M::CRITICS) {
    // ================================================================ critic wavefront: tiles wave - TILES, + CRITICS, ...
    if constexpr (AC) {
      const int j = lane & 15, gq = lane >> 4;
      TileNet<S, BF, REGW> net;
      net.init(packed_critic + run_off, smem + M::OFF_CRITIC, reinterpret_cast<const float*>(smem + M::OFF_CBIAS), lane);
      // values of the observations in the tiles of this wavefront -> dst [TE][N]
      auto values = [&](int parity, float* dst) {
        for (int c0 = (wave - TILES) * 16; c0 < B; c0 += M::CRITICS * 16) {
          float v[KS1][8];
#pragma unroll
          for (int s = 0; s < KS1; ++s) load_row_inputs<S>(obs_tile + (size_t(parity) * B + c0) * D, j, gq, s, v[s]);
          const f32x4 z = net.forward(v);
          if (gq == 0 && c0 + j < nvalid * N) dst[g0 * N + c0 + j] = (!BF && S::kRowTerms) ? (z[0] + z[1]) + z[2] : z[0];
        }
      };
      if (!head) __syncthreads();
      __syncthreads();
      float* value_p = A.value_traj ? A.value_traj + size_t(slot.t0) * TE * N : nullptr;
      for (int t = 0; t < slot.len; ++t) {
        __syncthreads();
        if (value_p) {   // of the observation that step t acted on
          values(t & 1, value_p);
          value_p += TE * N;
          if (t + 1 == slot.turn) value_p += size_t(slot.jump) * TE * N;
        }
      }
      __syncthreads();
      if (A.last_value && head) values(slot.len & 1, A.last_value);
    }
  } else {
    // ================================================================ service wavefront: rows 64 w .. of the block
    const int w = wave - TILES - M::CRITICS;
    const int r0 = w * 64;
    constexpr int kLastRows = B - (M::SERVICE - 1) * 64;                 // rows of the last service wavefront
    const bool has_row = M::SERVICE * 64 == B || r0 + lane < B;
    const int row = has_row ? r0 + lane : r0, el = row / N, i = row - el * N;
    const size_t g = g0 + el;
    const bool valid = has_row && g < TE;
    const uint32_t gc = g < TE ? uint32_t(g) : uint32_t(g0);
    const uint32_t run = gc / A.E, env = gc - run * A.E;
    const bool env_writer = valid && i == 0;
    const size_t row_off = size_t(gc) * N + i;
    const int my_rows = min(max(nvalid * N - r0, 0), min(64, B - r0));   // rows of this wavefront that exist
    [[maybe_unused]] float lx[L + 1], ly[L + 1];
#pragma unroll
    for (int k = 0; k < L + 1; ++k) lx[k] = ly[k] = 0.0f;
    int32_t ep = 0;
    if (g < TE) {
      if constexpr (!kTag) {
        if (head) {
#pragma unroll
          for (int k = 0; k < L; ++k) {
            lx[k] = A.st.pos_l[(0 * L + k) * TE + g];
            ly[k] = A.st.pos_l[(1 * L + k) * TE + g];
          }
        }
      }
      ep = A.st.ep_step[g];
    }
    if (SLOTS) counter_read(ep);
    [[maybe_unused]] const int32_t ep0 = ep;
    [[maybe_unused]] TagRole me{};
    if constexpr (kTag) me = tag_role<TS>(i, tg);
    uint32_t step = A.abs_step + uint32_t(slot.t0);

    // sampling noise of step `step` into the buffer of its parity
    auto draw_noise = [&](int parity, uint32_t at) {
      float nz[kNumActions];
      gumbel_noise(nz, A.seed, run, env, at, uint32_t(i));
      if (has_row) {
#pragma unroll
        for (int k = 0; k < kNumActions; ++k) noise[(parity * kNumActions + k) * B + row] = nz[k];
      }
    };
    auto flush = [&](int parity, float* slice) {   // this wavefront's rows to its slot of a [env][N][D] slice
      const float* src = obs_tile + (size_t(parity) * B + r0) * D;
      float* dst = slice + (g0 * N + r0) * D;
      const bool vec4 = (reinterpret_cast<uintptr_t>(dst) & 15u) == 0;
      if (vec4 && my_rows == 64) stream_out_full<64 * D / 4>(src, dst, lane);
      else if (vec4 && my_rows == kLastRows) stream_out_full<kLastRows * D / 4>(src, dst, lane);
      else stream_out(src, dst, my_rows * D, vec4, lane);
    };
    // the positions of an episode that starts at step `at` into the buffer of a parity
    auto draw_fresh = [&](int parity, uint32_t at) {
      uint32_t env_r = env;
      asm volatile("" : "+v"(env_r));
      float2* f = fresh + (size_t(parity) * EB + el) * M::ENT;
      // entities i, i + N, ... of the env (agents first, then landmarks)
#pragma unroll
      for (int e = 0; e < (M::ENT + N - 1) / N; ++e) {
        const int ent = i + e * N;
        if (ent < M::ENT) {
          const uint4 d = philox4x32_10(env_r, at, uint32_t(ent), kTagResetPos, A.seed, run);
          float2 p = make_float2(word_to_position(d.x), word_to_position(d.y));
          if (kTag && e > 0) { p.x *= 0.9f; p.y *= 0.9f; }   // obstacles start inside [-0.9, 0.9)
          if (has_row) f[ent] = p;
        }
      }
    };
    auto take_landmarks = [&](int parity) {
      const float2* f = fresh + (size_t(parity) * EB + el) * M::ENT;
#pragma unroll
      for (int k = 0; k < L; ++k) {
        lx[k] = f[N + k].x;
        ly[k] = f[N + k].y;
      }
    };
    const bool per_agent = kTag || A.ph.reward_mode == 1;
    float* obs_p = A.obs_traj;
    uint8_t* act_p = A.act_traj;
    float* rew_p = A.rew_traj;
    uint8_t* done_p = A.done_traj;
    [[maybe_unused]] float* logp_p = A.logp_traj;
    auto advance = [&](int steps) {
      const size_t envs = size_t(steps) * TE;
      if (obs_p) obs_p += envs * (N * D);
      if (act_p) act_p += envs * N;
      if (rew_p) rew_p += per_agent ? envs * N : envs;
      if (done_p) done_p += envs;
      if (AC && logp_p) logp_p += envs * N;
    };

    draw_noise(0, step);
    if (!head) {
      advance(slot.t0);
      draw_fresh(1, step);
      ep = 0;
      __syncthreads();
      if constexpr (!kTag) take_landmarks(1);
    }
    __syncthreads();
    [[maybe_unused]] uint32_t ticket = 0;
    if (SLOTS && env_writer) ticket = take_ticket(A, g);
    for (int t = 0; t < slot.len; ++t) {
      const int par = t & 1;
      const bool turn = t + 1 == slot.turn;
      const uint32_t next = step + 1u + (turn ? uint32_t(slot.jump) : 0u);
      // ---- ahead: noise of step t + 1, and the new episode's draw if this env's ends with step t
      draw_noise(par ^ 1, next);
      const bool done = ep + 1 >= max_ep;
      if (done) draw_fresh(par, next);
      __syncthreads();
      // ---- behind: everything that leaves the chip for step t
      if (obs_p) {
        flush(par, obs_p);
        obs_p += TE * (N * D);
      }
      const uint32_t act = acts[par * B + row];
      if (act_p) {
        if (valid) act_p[row_off] = uint8_t(act);
        act_p += TE * N;
      }
      if constexpr (AC) {
        if (logp_p) {
          // log pi(act | obs) = z_act - max - ln sum exp(z - max)
          float z[kNumActions];
#pragma unroll
          for (int k = 0; k < kNumActions; ++k) z[k] = logits[(par * kNumActions + k) * B + row];
          float zmax = z[0], zact = z[0];
#pragma unroll
          for (int k = 1; k < kNumActions; ++k) {
            zmax = fmaxf(zmax, z[k]);
            zact = act == uint32_t(k) ? z[k] : zact;
          }
          float sum = 0.0f;
#pragma unroll
          for (int k = 0; k < kNumActions; ++k) sum += hw_exp2((z[k] - zmax) * kLog2e);
          if (valid) logp_p[row_off] = (zact - zmax) - kLn2 * hw_log2(sum);
          logp_p += TE * N;
        }
      }
      if (rew_p) {
        float qx[N], qy[N];
#pragma unroll
        for (int a = 0; a < N; ++a) {
          const float4 p = xch[par * B + el * N + a];
          qx[a] = p.x;
          qy[a] = p.y;
        }
        float px = 0.0f, py = 0.0f;
#pragma unroll
        for (int a = 0; a < N; ++a) {
          if (a == i) { px = qx[a]; py = qy[a]; }
        }
        if constexpr (kTag) {
          const float r = tag_reward<TS>(i, me, tg, px, py, qx, qy);
          if (valid) rew_p[row_off] = r;
        } else {
          const float r = coverage_reward(qx, qy, lx, ly);
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
      ep = done ? 0 : ep + 1;
      if constexpr (!kTag) {
        if (done) take_landmarks(par);
      }
      step = next;
      if (turn) advance(slot.jump);
    }
    __syncthreads();
    if (A.last_obs && head) flush(slot.len & 1, A.last_obs);
    if (SLOTS && env_writer) settle_ticket(A, max_ep, g, ticket, ep0);
  }
}

template <typename Scn, int EB, bool AC, bool BF, bool REGW, int MINW>
hipError_t launch_small_impl(const TagArgs& A, const void* packed, const void* critic, hipStream_t s) {
  using M = SmallSmem<Scn, EB, AC, BF, REGW>;
  static std::atomic<uint64_t> lds_allowed[2];
  const uint32_t groups = (A.r.TE + EB - 1) / EB;
  auto launch = [&](auto kern, dim3 grid, auto piece) {
    hipLaunchKernelGGL(kern, grid, dim3(M::WAVES * 64), M::TOTAL, s, A, static_cast<const uint8_t*>(packed),
                       static_cast<const uint8_t*>(critic), int(A.r.TE != A.r.E), piece);
  };
  if (A.r.slots > 1) {
    auto kern = rollout_small_kernel<Scn, EB, AC, BF, REGW, MINW, SlotGrid>;
    if (hipError_t e = allow_lds(reinterpret_cast<const void*>(kern), M::TOTAL, lds_allowed[1]); e != hipSuccess) return e;
    launch(kern, slots_grid(A.r, groups), SlotGrid{groups});
    return hipGetLastError();
  }
  auto kern = rollout_small_kernel<Scn, EB, AC, BF, REGW, MINW, GridPiece>;
  if (hipError_t e = allow_lds(reinterpret_cast<const void*>(kern), M::TOTAL, lds_allowed[0]); e != hipSuccess) return e;
  return launch_groups<M::WAVES * 64>(groups, [&](dim3 grid, const GridPiece& p) { launch(kern, grid, p); });
}

// ALONE: every block has a CU to itself
template <typename Scn, int EB, bool AC, bool BF, bool ALONE = false>
hipError_t launch_small_eb(const TagArgs& A, const void* packed, const void* critic, hipStream_t s) {
  // Stationary operands while a block has a CU to itself (6-10 % faster there); they take 100 to 170 registers per
  // wavefront, so beyond that, and with more than 8 wavefronts per block, the operands are read from LDS.
  constexpr int W = SmallSmem<Scn, EB, AC, BF, true>::WAVES, kMin = (W + 3) / 4;
  if constexpr (kMin <= 2) {
    if constexpr (ALONE) return launch_small_impl<Scn, EB, AC, BF, true, 2>(A, packed, critic, s);
    if ((A.r.TE + EB - 1) / EB * uint32_t(A.r.slots) <= compute_units()) return launch_small_impl<Scn, EB, AC, BF, true, 2>(A, packed, critic, s);
  }
  if constexpr (!ALONE || kMin > 2) return launch_small_impl<Scn, EB, AC, BF, false, (kMin < 4 ? 4 : kMin)>(A, packed, critic, s);
}

// *taken: whether the rollout was launched here.  unfit: runs that suit no block of the other kernels, which the caller
// knows; they always come here (1,024 runs x 16 envs x 3 agents 473 us against 596 in the 16-env blocks of half-filled
// wavefronts that such runs used before, actor-critic 883 against 2,044; predator-prey: see run_blocks16 in mpe_tag.hip).
template <typename Scn, bool AC, bool BF>
hipError_t launch_small(const TagArgs& A, bool unfit, const void* packed, const void* critic, hipStream_t s, bool* taken) {
  constexpr int N = Scn::N;
  constexpr uint32_t kWavesBlock = waves_block_envs(N);
  // Blocks are 16 envs, the paper's run size (16 envs x N agents are N whole tiles); 8 envs with 6, 8 and 10 agents while
  // such blocks have a CU each (actor-critic, 2,048 envs: 8 agents 507 against 817 us, predator-prey with 10 agents 600
  // against 1,044), and where the rows and both networks of 16 envs x 10 agents pass the LDS.
  constexpr bool kEight = N == 6 || N == 8 || N == 10, kOnlyEight = AC && N == 10 && Scn::D > 32;
  const bool runs = A.r.TE != A.r.E;
  if (runs && A.r.E % 16 != 0) return hipSuccess;
  if (A.r.slots > 1 && !slots_fit(A.r, kOnlyEight ? 8 : 16)) return hipSuccess;
  const uint32_t cus = compute_units(), blocks16 = (A.r.TE + 15) / 16 * uint32_t(A.r.slots);
  if (!(runs && unfit)) {
    constexpr SmallRange one = small_range<Scn::kTag, N, AC, BF>(), several = small_range_slots<Scn::kTag, N, AC, BF>();
    const SmallRange range = A.r.slots > 1 ? several : one;
    const bool first_round_full = A.r.work() > kWavesBlock * cus;
    // One agent's blocks are two or three wavefronts around 33 KB of weights per network: in a rollout of one step the
    // staging of a full range of them is what counts (32,768 envs 11.4 us, 64-env blocks 8.3; actor-critic 22.1 against 17.3).
    const uint32_t upto = N == 1 && A.r.T == 1 ? 70 : range.upto;
    if (blocks16 * 10 > cus * (first_round_full && range.past ? range.past : upto)) return hipSuccess;
    constexpr BatchKind kind{N, Scn::kTag, BF, AC};
    if (A.r.slots > 1 && !slots_pay(A.r, small_time(kind, A.r), one_slot_time(kind, A.r, one.upto))) return hipSuccess;
  }
  *taken = true;
  if constexpr (kEight) {
    if (kOnlyEight || (A.r.TE + 7) / 8 * uint32_t(A.r.slots) <= cus) return launch_small_eb<Scn, 8, AC, BF, !kOnlyEight>(A, packed, critic, s);
  }
  if constexpr (!kOnlyEight) return launch_small_eb<Scn, 16, AC, BF>(A, packed, critic, s);
}

}  // namespace

}  // namespace mpe
