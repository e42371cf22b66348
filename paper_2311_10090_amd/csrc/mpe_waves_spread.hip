// Full-batch fused rollout with independent wavefronts, simple spread: 3 to 10 agents, fp32 weights.
#include "mpe_waves.h"

namespace mpe {

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

}  // namespace mpe
