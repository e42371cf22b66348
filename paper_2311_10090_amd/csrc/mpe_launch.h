// Host-side launch interface between the C ABI (mpe_api.hip) and the kernel files.
#pragma once

#include <atomic>

#include "mpe_device.h"

namespace mpe {

// A kernel that needs more than 64 KB of dynamic LDS must be allowed to, once per device it is
// launched on (function attributes belong to the device's copy of the code).  `done` holds one bit
// per device ordinal; setting the attribute twice from two threads is harmless.
inline hipError_t allow_lds(const void* kern, size_t bytes, std::atomic<uint64_t>& done) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = 1ull << (unsigned(dev) & 63u);
  if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
  e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
  if (e == hipSuccess) done.fetch_or(bit, std::memory_order_release);
  else (void)hipGetLastError();   // reported here, not by a later launch's check
  return e;
}

// Compute units of the current device (queried once per process; launch shapes are chosen by it).
inline uint32_t compute_units() {
  static std::atomic<int> cus{0};
  int n = cus.load(std::memory_order_relaxed);
  if (n == 0) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
      n = 256;
    cus.store(n, std::memory_order_relaxed);
  }
  return uint32_t(n);
}

// Blocks of the kernels with one or more lanes per agent, each of which steps one group of envs.
// The hardware deals block b to XCD b % 8; each XCD gets one contiguous range of groups, so that the partial cache lines
// which neighbouring groups write per step meet in one L2.
// A grid dimension holds fewer than 2^32 threads, which these kernels need at 2.0e8 to 1.1e9 envs (the two wavefronts of 6
// envs x 10 agents: 21 threads per env): groups beyond 2^31 threads go to further launches.
struct GridPiece {
  uint32_t first, end, per_xcd;   // groups [first, end)
};
__device__ __forceinline__ uint32_t xcd_group(const GridPiece& p) {   // not below p.end for a block that is left over
  return p.first + (blockIdx.x & 7u) * p.per_xcd + (blockIdx.x >> 3);
}
template <int THREADS, typename Launch>
hipError_t launch_groups(uint32_t groups, Launch launch) {
  constexpr uint32_t kPiece = (1u << 31) / uint32_t(THREADS) / 8u * 8u;
  for (uint32_t first = 0; first < groups; first += kPiece) {
    const uint32_t n = groups - first < kPiece ? groups - first : kPiece, per_xcd = (n + 7) / 8;
    launch(dim3(per_xcd * 8), GridPiece{first, first + n, per_xcd});
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  }
  return hipSuccess;
}

struct RolloutArgs {
  StatePtrs st;
  Phys ph;
  uint32_t TE;        // total envs = runs * envs per run
  uint32_t E;         // envs per run
  uint32_t seed;
  uint32_t abs_step;  // absolute step of the first transition
  int32_t T;
  float* obs_traj;    // [T][TE][N][D] or null
  uint8_t* act_traj;  // [T][TE][N]    or null
  float* rew_traj;    // [T][TE]       or null
  uint8_t* done_traj; // [T][TE]       or null
  float* last_obs;    // [TE][N][D]    or null
  // actor-critic rollout only (null otherwise)
  float* logp_traj = nullptr;   // [T][TE][N] log-probability of the sampled action
  float* value_traj = nullptr;  // [T][TE][N] critic value of the observation acted on
  float* last_value = nullptr;  // [TE][N]    critic value of last_obs
  // Word that a kernel raises (system scope) when a bounded wait gave up; null = not reported.
  uint32_t* fault = nullptr;
  // Polls after which a wait at a sync-group barrier gives up (kBarrierSpinLimit unless a test lowers it).
  uint32_t barrier_polls = 1u << 24;
  // Slots of time that run side by side, steps of one (mpe_slots.h).
  int32_t slots = 1, span = 0;
  // Blocks of which envs, from the first one on, have their episode counters alike: of this many, or a part of it (counter_unit); 0: any.  For the
  // host alone, and where the struct had padding: the kernels' arguments, and so their code, are as without it.
  uint32_t alike = 0;
  uint32_t work() const { return TE * uint32_t(slots); }   // envs that the launch steps side by side
};

// Predator-prey scenario: constants by role (index 0 adversary, 1 good agent), combined on the
// host in double and rounded once.
struct TagPhys {
  float dt, keep, dt_over_mass, inv_margin, force_margin;
  int32_t max_ep;
  float radius[2];
  float gain[2];
  float limit[2];      // speed limit
  float limit_sq[2];
  float lm_radius;
  float touch_sq;      // (adversary radius + good radius)^2
};

struct TagArgs {
  RolloutArgs r;                 // state, sizes, seed, step, outputs (r.ph is unused)
  TagPhys tg;
  const uint8_t* actions_in;     // [TE][N], single step with given actions only (launch_env_agents)
};

// Every launch function returns what the runtime said of the launch, and hipErrorInvalidValue (nothing launched) for a
// shape that it is not built for.

// The predator-prey shapes that are built: (agents, landmarks, good agents).
#define MPE_TAG_SHAPES(X) X(4, 2, 1) X(2, 1, 1) X(3, 0, 1) X(6, 2, 2) X(5, 2, 1) X(8, 2, 2) X(10, 3, 2)

// (N, L, G) = agents, landmarks, good agents
bool tag_supported(int N, int L, int G);
bool tag_policy_supported(int N, int L, int G, int H, int weight_dtype);
hipError_t launch_tag_reset(int N, int L, int G, const StatePtrs& st, uint32_t TE, uint32_t E, uint32_t seed, float* obs,
                            hipStream_t s);
// mode 1: uniform random actions; mode 2: the packed fp32 policy;
// mode 3: the packed bf16 policy; mode 4 / 5: the packed fp32 / bf16 policy and critic (actor-critic outputs in r)
hipError_t launch_tag_rollout(int N, int L, int G, int mode, const TagArgs& A, const void* packed,
                              const void* packed_critic, hipStream_t s, const char** why);
struct PolicyBuffers;
// nout: outputs of the last layer (5 policy logits, 1 critic value)
hipError_t pack_policy_tag(PolicyBuffers& pb, int N, int L, int G, int R, bool bf16, int nout, const float* W1,
                           const float* b1, const float* W2, const float* b2, const float* W3, const float* b3,
                           hipStream_t s);

hipError_t launch_reset(int N, const StatePtrs& st, uint32_t TE, uint32_t E, uint32_t seed, float* obs,
                        hipStream_t s);
// For mpe_set_state: no ticket is taken, and unit[0 ..] = the units of the counters' stretches (counter_unit), one per block.
constexpr uint32_t kCounterBlocks = 256;
inline uint32_t counter_blocks(uint32_t TE) { return TE / 1024 < kCounterBlocks ? TE / 1024 + 1 : kCounterBlocks; }
hipError_t launch_read_counters(const StatePtrs& st, uint32_t TE, uint32_t* unit, hipStream_t s);
hipError_t launch_step(int N, const StatePtrs& st, const Phys& ph, uint32_t TE, uint32_t E, uint32_t seed,
                       uint32_t abs_step, const uint8_t* actions, float* obs, float* reward, uint8_t* done,
                       hipStream_t s);
hipError_t launch_rollout_uniform(int N, const RolloutArgs& A, hipStream_t s);

// Policy weights re-packed into MFMA A-operand order (device memory owned by the handle, or, `borrowed`,
// a piece of memory of `bytes` bytes that is never freed or grown here).
struct PolicyBuffers {
  void* packed = nullptr;
  size_t bytes = 0;
  bool borrowed = false;
};
// Bytes that pack_policy writes for R runs (0 for an unsupported shape).
size_t packed_policy_bytes(int N, int H, int R, int weight_dtype);

// Both return a HIP status; *why is set (and nothing launched) when the shape is unsupported.
hipError_t pack_policy(PolicyBuffers& pb, int N, int H, int R, int weight_dtype, const float* W1,
                       const float* b1, const float* W2, const float* b2, const float* W3,
                       const float* b3, hipStream_t s, const char** why);
hipError_t launch_rollout_policy(int N, int H, int weight_dtype, const RolloutArgs& A,
                                 const PolicyBuffers& pb, hipStream_t s, const char** why);
void free_policy(PolicyBuffers& pb);

// Per-kernel-family entry points behind pack_policy / launch_rollout_policy.
bool wide_supported(int N, int H);                       // bf16 general kernel
size_t packed_run_bytes_wide(int N, int H);
hipError_t pack_policy_wide(PolicyBuffers& pb, int N, int H, int R, const float* W1, const float* b1,
                            const float* W2, const float* b2, const float* W3, const float* b3, int nout,
                            hipStream_t s);
hipError_t launch_rollout_ac_wide(int N, int H, const RolloutArgs& A, const PolicyBuffers& pb,
                                  const PolicyBuffers& critic, hipStream_t s, const char** why);
hipError_t launch_rollout_policy_wide(int N, int H, const RolloutArgs& A, const PolicyBuffers& pb, hipStream_t s,
                                      const char** why);
hipError_t launch_rollout_uniform_wide(int N, const RolloutArgs& A, hipStream_t s);
bool f32_supported(int N, int H, bool bf16);             // headline kernel (H = 64; N <= 3, with fp32 weights N <= 10)
size_t packed_run_bytes_f32(int N, bool bf16);
hipError_t pack_policy_f32(PolicyBuffers& pb, int N, int R, const float* W1, const float* b1, const float* W2,
                           const float* b2, const float* W3, const float* b3, int nout, bool bf16, hipStream_t s);
hipError_t launch_rollout_ac_f32(int N, bool bf16, const RolloutArgs& A, const PolicyBuffers& pb,
                                 const PolicyBuffers& critic, hipStream_t s, const char** why);
hipError_t launch_rollout_policy_f32(int N, bool bf16, const RolloutArgs& A, const PolicyBuffers& pb, hipStream_t s,
                                     const char** why);
hipError_t ensure_policy_bytes(PolicyBuffers& pb, size_t bytes);

// Recurrent policy (hidden 128, bf16): simple spread with 1..10 agents.
// tag: the predator-prey scenario with (N, L, G) agents, landmarks, good agents; otherwise simple spread (L, G unused)
bool gru_supported(bool tag, int N, int L, int G, int H, int weight_dtype);
// D = observation width of the scenario, TE, E = all envs, envs per run
hipError_t pack_policy_gru(PolicyBuffers& pb, bool tag, int N, int D, uint32_t TE, uint32_t E, const float* We, const float* be, const float* Wi,
                           const float* bi, const float* Wh, const float* bh, const float* Wf, const float* bf,
                           const float* Wo, const float* bo, hipStream_t s);
// hidden: [TE][N][128] fp32, read at the start and written at the end of the rollout; A.tg is read by the
// predator-prey shapes only
// critic: the packed critic head (pack_gru_critic) for the actor-critic rollout (A.r.logp_traj, value_traj,
// last_value), or null for the plain one
// *partial: the launch of a part of the batch failed after that of another, which runs (state and hidden are then no step's)
hipError_t launch_rollout_gru(bool tag, int N, int L, int G, const TagArgs& A, const PolicyBuffers& pb, const void* critic,
                              float* hidden, hipStream_t s, bool* partial, const char** why);
// Critic head of the recurrent actor-critic: Wc [R][128][128], bc [R][128], wv [R][128], bv [R]
hipError_t pack_gru_critic(PolicyBuffers& pb, uint32_t TE, uint32_t E, const float* Wc, const float* bc, const float* wv,
                           const float* bv, hipStream_t s);
// One lane per agent (mpe_env_agents.hip), both scenarios: one step under A.actions_in (reward, done and obs after the
// step through A.r.rew_traj, done_traj, last_obs), or, with A.actions_in null, a rollout with uniform actions.
// Envs in a block of it.
constexpr uint32_t env_agents_block(int N) { return uint32_t(64 / N / 2 * 2); }
// Whether its rollout is the faster one for this batch.
bool env_agents_faster(bool tag, int N, uint32_t TE);
// The most slots of time (mpe_slots.h) that its rollout, or for up to 3 agents of simple spread that of mpe_env_kernels.hip, is to use.
uint32_t env_slots(bool tag, int N, int D, uint32_t TE);
hipError_t launch_env_agents(bool tag, int N, int L, int G, const TagArgs& A, hipStream_t s);
// Blocks of half-filled wavefronts are up to 16 threads per env and launched whole: for up to this many envs, 2^31 threads.
constexpr uint32_t kWholeLaunchEnvs = 1u << 27;
// Envs in the smallest block of the independent wavefronts: 4 of them, each of as many whole envs as fit its 64 lanes.
constexpr uint32_t waves_block_envs(uint32_t N) { return 4 * (64 / N); }
// Several runs that would fill less than half of such a block.
inline bool half_empty_waves(const RolloutArgs& A, uint32_t N) { return A.TE != A.E && A.E * 2 < waves_block_envs(N); }
// Full batches, independent wavefronts (mpe_waves.h).  critic: the packed critic of the actor-critic rollout, or null.
hipError_t launch_waves_spread(int N, bool bf16, const TagArgs& A, const void* packed, const void* critic, hipStream_t s);
hipError_t launch_waves_tag(int N, int L, int G, bool bf16, const TagArgs& A, const void* packed, const void* critic, hipStream_t s);
// The same in the slots of A (mpe_slots.h): *taken = true and launched where that pays.
hipError_t launch_waves_spread_slots(int N, bool bf16, const TagArgs& A, const void* packed, const void* critic, hipStream_t s, bool* taken);
// against: this kernel would also run the batch in one slot
hipError_t launch_waves_tag_slots(int N, int L, int G, bool bf16, const TagArgs& A, bool against, const void* packed, const void* critic,
                                  hipStream_t s, bool* taken);
// Small batches and small runs (mpe_small.h): *taken = true and the rollout launched where that kernel is the faster
// one for the batch, else nothing done.  A.tg is read by the predator-prey shapes only.
// unfit: the runs suit no block of the other kernels.
hipError_t launch_small_spread(int N, bool bf16, const TagArgs& A, bool unfit, const void* packed, hipStream_t s, bool* taken);
hipError_t launch_small_spread_ac(int N, bool bf16, const TagArgs& A, bool unfit, const void* packed, const void* critic,
                                  hipStream_t s, bool* taken);
hipError_t launch_small_tag(int N, int L, int G, bool bf16, const TagArgs& A, bool unfit, const void* packed, hipStream_t s,
                            bool* taken);
hipError_t launch_small_tag_ac(int N, int L, int G, bool bf16, const TagArgs& A, bool unfit, const void* packed,
                               const void* critic, hipStream_t s, bool* taken);
hipError_t launch_fill_zero(float* p, size_t n, hipStream_t s);

}  // namespace mpe
