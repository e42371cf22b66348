// Small-batch fused rollout, predator-prey: every shape, fp32 or bf16 weights.
#include "mpe_small.h"

namespace mpe {

hipError_t launch_small_tag(int N, int L, int G, bool bf16, const TagArgs& A, bool unfit, const void* packed, hipStream_t s, bool* taken) {
#define X(n, l, g)                                                                             \
  if (N == n && L == l && G == g)                                                              \
    return bf16 ? launch_small<SmallTag<n, l, g>, false, true>(A, unfit, packed, nullptr, s, taken)     \
                : launch_small<SmallTag<n, l, g>, false, false>(A, unfit, packed, nullptr, s, taken);
  MPE_TAG_SHAPES(X)
#undef X
  return hipErrorInvalidValue;
}

}  // namespace mpe
