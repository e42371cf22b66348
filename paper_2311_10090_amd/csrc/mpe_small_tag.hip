// Small-batch fused rollout, predator-prey: every shape, fp32 or bf16 weights.
#include "mpe_small.h"

namespace mpe {

#define MPE_SMALL_TAG_SHAPES(X) X(4, 2, 1) X(2, 1, 1) X(3, 0, 1) X(6, 2, 2) X(5, 2, 1) X(8, 2, 2) X(10, 3, 2)

hipError_t launch_small_tag(int N, int L, int G, bool bf16, const TagArgs& A, uint32_t run_block, const void* packed, hipStream_t s, bool* taken) {
#define X(n, l, g)                                                                             \
  if (N == n && L == l && G == g)                                                              \
    return bf16 ? launch_small<SmallTag<n, l, g>, false, true>(A, run_block, packed, nullptr, s, taken)     \
                : launch_small<SmallTag<n, l, g>, false, false>(A, run_block, packed, nullptr, s, taken);
  MPE_SMALL_TAG_SHAPES(X)
#undef X
  return hipSuccess;
}


}  // namespace mpe
