// Small-batch fused rollout, simple spread, actor-critic: 1 to 10 agents with fp32 weights, 1 to 3 with bf16 ones.
#include "mpe_small.h"

namespace mpe {

hipError_t launch_small_spread_ac(int N, bool bf16, const TagArgs& A, bool unfit, const void* packed, const void* critic, hipStream_t s, bool* taken) {
  switch (N) {
    case 1: return bf16 ? launch_small<SmallSpread<1>, true, true>(A, unfit, packed, critic, s, taken)
                         : launch_small<SmallSpread<1>, true, false>(A, unfit, packed, critic, s, taken);
    case 2: return bf16 ? launch_small<SmallSpread<2>, true, true>(A, unfit, packed, critic, s, taken)
                         : launch_small<SmallSpread<2>, true, false>(A, unfit, packed, critic, s, taken);
    case 3: return bf16 ? launch_small<SmallSpread<3>, true, true>(A, unfit, packed, critic, s, taken)
                         : launch_small<SmallSpread<3>, true, false>(A, unfit, packed, critic, s, taken);
    case 4: return launch_small<SmallSpread<4>, true, false>(A, unfit, packed, critic, s, taken);
    case 5: return launch_small<SmallSpread<5>, true, false>(A, unfit, packed, critic, s, taken);
    case 6: return launch_small<SmallSpread<6>, true, false>(A, unfit, packed, critic, s, taken);
    case 7: return launch_small<SmallSpread<7>, true, false>(A, unfit, packed, critic, s, taken);
    case 8: return launch_small<SmallSpread<8>, true, false>(A, unfit, packed, critic, s, taken);
    case 9: return launch_small<SmallSpread<9>, true, false>(A, unfit, packed, critic, s, taken);
    case 10: return launch_small<SmallSpread<10>, true, false>(A, unfit, packed, critic, s, taken);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace mpe
