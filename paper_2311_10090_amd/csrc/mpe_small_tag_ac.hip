// Small-batch fused rollout, predator-prey, actor-critic: every shape, fp32 or bf16 weights.
#include "mpe_small.h"

namespace mpe {

hipError_t launch_small_tag_ac(int N, int L, int G, bool bf16, const TagArgs& A, bool unfit, const void* packed, const void* critic, hipStream_t s, bool* taken) {
#define X(n, l, g)                                                                             \
  if (N == n && L == l && G == g)                                                              \
    return bf16 ? launch_small<SmallTag<n, l, g>, true, true>(A, unfit, packed, critic, s, taken)     \
                : launch_small<SmallTag<n, l, g>, true, false>(A, unfit, packed, critic, s, taken);
  MPE_TAG_SHAPES(X)
#undef X
  return hipErrorInvalidValue;
}

}  // namespace mpe
