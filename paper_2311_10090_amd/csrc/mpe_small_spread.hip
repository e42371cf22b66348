// Small-batch fused rollout, simple spread: 1 to 10 agents with fp32 weights, 1 to 3 with bf16 ones.
#include "mpe_small.h"

namespace mpe {

hipError_t launch_small_spread(int N, bool bf16, const TagArgs& A, bool unfit, const void* packed, hipStream_t s, bool* taken) {
  switch (N) {
    case 1: return bf16 ? launch_small<SmallSpread<1>, false, true>(A, unfit, packed, nullptr, s, taken)
                         : launch_small<SmallSpread<1>, false, false>(A, unfit, packed, nullptr, s, taken);
    case 2: return bf16 ? launch_small<SmallSpread<2>, false, true>(A, unfit, packed, nullptr, s, taken)
                         : launch_small<SmallSpread<2>, false, false>(A, unfit, packed, nullptr, s, taken);
    case 3: return bf16 ? launch_small<SmallSpread<3>, false, true>(A, unfit, packed, nullptr, s, taken)
                         : launch_small<SmallSpread<3>, false, false>(A, unfit, packed, nullptr, s, taken);
    case 4: return launch_small<SmallSpread<4>, false, false>(A, unfit, packed, nullptr, s, taken);
    case 5: return launch_small<SmallSpread<5>, false, false>(A, unfit, packed, nullptr, s, taken);
    case 6: return launch_small<SmallSpread<6>, false, false>(A, unfit, packed, nullptr, s, taken);
    case 7: return launch_small<SmallSpread<7>, false, false>(A, unfit, packed, nullptr, s, taken);
    case 8: return launch_small<SmallSpread<8>, false, false>(A, unfit, packed, nullptr, s, taken);
    case 9: return launch_small<SmallSpread<9>, false, false>(A, unfit, packed, nullptr, s, taken);
    case 10: return launch_small<SmallSpread<10>, false, false>(A, unfit, packed, nullptr, s, taken);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace mpe
