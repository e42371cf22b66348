// Full-batch fused rollout with independent wavefronts, simple spread: 1 to 10 agents with fp32 weights, 1 to 3 with bf16 ones.
#include "mpe_waves.h"

namespace mpe {

// one slot: 3 to 10 agents, fp32
hipError_t launch_waves_spread(int N, bool bf16, const TagArgs& A, const void* packed, const void* critic, hipStream_t s) {
  if (bf16) return hipErrorInvalidValue;
#define X(n)                                                                                     \
  case n: return critic ? launch_waves<WaveSpread<n>, true, false>(A, packed, critic, s)         \
                        : launch_waves<WaveSpread<n>, false, false>(A, packed, nullptr, s);
  switch (N) {
    X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10)
    default: return hipErrorInvalidValue;
  }
#undef X
}

hipError_t launch_waves_spread_slots(int N, bool bf16, const TagArgs& A, const void* packed, const void* critic, hipStream_t s, bool* taken) {
#define X(n, bf)                                                                                                       \
  case n: return critic ? launch_waves_slots<WaveSpread<n>, true, bf>(A, n > 3, packed, critic, s, taken)              \
                        : launch_waves_slots<WaveSpread<n>, false, bf>(A, n > 3, packed, nullptr, s, taken);
  if (bf16) {
    switch (N) {
      X(1, true) X(2, true) X(3, true)
      default: return hipErrorInvalidValue;
    }
  }
  switch (N) {
    X(1, false) X(2, false) X(3, false) X(4, false) X(5, false) X(6, false) X(7, false) X(8, false) X(9, false) X(10, false)
    default: return hipErrorInvalidValue;
  }
#undef X
}

}  // namespace mpe
