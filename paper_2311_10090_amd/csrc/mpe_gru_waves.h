// Weight image of the recurrent rollout's independent wavefronts (mpe_gru_waves.hip; packed by mpe_policy_gru.hip with the other one)
// and the host-side interface to them.
#pragma once

#include "mpe_launch.h"

namespace mpe {

// Bytes of the images of the other recurrent kernel, behind which (one run) these follow: see mpe_policy_gru.hip.
constexpr size_t kGruImageBytes = (16 + 8 * 24 + 32 + 4) * 1024 + size_t(6 * 128 + 16) * 4;
constexpr size_t kGruCriticImageBytes = 32 * 1024 + size_t(2 * 128 + 4) * 4;

// A operands of v_mfma_f32_16x16x32_bf16, 1 KB each, lane (row = lane % 16, gq = lane / 16) holds weights
// [32 s + 8 gq + e][unit of row], e = 0..7:
//   the 192 operands of the gates are consumed in a fixed order (gate_part): per unit tile c, n recurrent 4 K slices, r 8,
//   n input 4, z 8; three of four are staged in LDS ([RESIDENT]), every fourth is read from the image each step
//   [RESIDENT] | embedding [c 8][s kse] | gates, every fourth [48] | second layer [c 8][s 4] | outputs [s 4] |
//   fp32 biases: embedding, r, z, n input, n recurrent, second layer [128 each], outputs [16]
// The rows of a pair of unit tiles are permuted (unit) so that the accumulators of a layer are, as they lie, the B operands of
// the next in natural K order: the sums are those of the block kernel (mpe_policy_gru.hip) bit for bit.  (A matrix
// instruction adds its products eight at a time, one lane group after the other: another order of K inside a slice
// rounds differently, checked on the chip.)
struct GruWavePk {
  static constexpr int kG = 128, kFrag = 1024, RESIDENT = 144, BIAS_FLOATS = 6 * kG + 16;
  __host__ __device__ static constexpr size_t base() { return kGruImageBytes; }
  __host__ __device__ static constexpr int frags(int kse) { return RESIDENT + 8 * kse + 48 + 32 + 4; }
  __host__ __device__ static constexpr size_t bytes(int kse) { return size_t(frags(kse)) * kFrag + BIAS_FLOATS * 4; }
  // unit of row r of unit tile c: accumulator q of lane group gq is row 4 gq + q
  __host__ __device__ static constexpr int unit(int c, int r) { return 32 * (c / 2) + 8 * (r / 4) + 4 * (c % 2) + r % 4; }
  // gate operand q (0..23) of a unit tile: n recurrent, then r with input and recurrent slices in turn (the block kernel's
  // order), n input, z like r
  struct Part { int gate, recurrent, s; };      // gate 0 r, 1 z, 2 n
  __host__ __device__ static constexpr Part gate_part(int q) {
    if (q < 4) return {2, 1, q};
    if (q < 12) return {0, (q - 4) % 2, (q - 4) / 2};
    if (q < 16) return {2, 0, q - 12};
    return {1, (q - 16) % 2, (q - 16) / 2};
  }
  // output of row r of the last layer: 0..3 in lane groups 0 and 2, output 4 in the first row of groups 1 and 3
  __host__ __device__ static constexpr int out_row(int r) { return r % 8 < 4 ? r % 4 : (r % 8 == 4 ? 4 : -1); }
};
// Critic head: second layer [c 8][s 4] | fp32: its biases [128], value weights rounded to bf16 [128], output bias
struct GruWaveCriticPk {
  static constexpr int FRAGS = 32, BIAS_FLOATS = 2 * 128 + 4;
  __host__ __device__ static constexpr size_t base() { return kGruCriticImageBytes; }
  static constexpr size_t BYTES = size_t(FRAGS) * 1024 + BIAS_FLOATS * 4;
};

// Envs in a block: 8 wavefronts of 32 rows.
constexpr uint32_t gru_waves_block_envs(int N) { return 8u * (32u / uint32_t(N)); }

// The first `envs` envs of the batch; in several slots of time (A.r.slots) the envs of all slots, which is the whole batch.
hipError_t launch_gru_waves(bool tag, int N, int L, int G, const TagArgs& A, const void* packed, const void* critic, float* hidden,
                            uint32_t envs, hipStream_t s);

}  // namespace mpe
