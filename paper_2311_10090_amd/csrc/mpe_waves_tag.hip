// Full-batch fused rollout with independent wavefronts, predator-prey.
#include "mpe_waves.h"

namespace mpe {

hipError_t launch_waves_tag(int N, int L, int G, bool bf16, const TagArgs& A, const void* packed, const void* critic, hipStream_t s) {
  // one slot, 3 agents: the actor-critic rollout only (the plain one is mpe_tag.hip's at every size)
  if (N == 3 && L == 0 && G == 1) {
    if (!critic) return hipErrorInvalidValue;
    return bf16 ? launch_waves<WaveTag<3, 0, 1>, true, true>(A, packed, critic, s)
                : launch_waves<WaveTag<3, 0, 1>, true, false>(A, packed, critic, s);
  }
#define X(n, l, g)                                                                                                  \
  if (N == n && L == l && G == g) {                                                                                 \
    if (bf16)                                                                                                       \
      return critic ? launch_waves<WaveTag<n, l, g>, true, true>(A, packed, critic, s)                              \
                    : launch_waves<WaveTag<n, l, g>, false, true>(A, packed, nullptr, s);                           \
    return critic ? launch_waves<WaveTag<n, l, g>, true, false>(A, packed, critic, s)                               \
                  : launch_waves<WaveTag<n, l, g>, false, false>(A, packed, nullptr, s);                            \
  }
  X(4, 2, 1) X(6, 2, 2) X(5, 2, 1) X(8, 2, 2) X(10, 3, 2)
#undef X
  return hipErrorInvalidValue;
}

hipError_t launch_waves_tag_slots(int N, int L, int G, bool bf16, const TagArgs& A, bool against, const void* packed, const void* critic,
                                  hipStream_t s, bool* taken) {
#define X(n, l, g)                                                                                                        \
  if (N == n && L == l && G == g) {                                                                                       \
    if (bf16)                                                                                                             \
      return critic ? launch_waves_slots<WaveTag<n, l, g>, true, true>(A, against, packed, critic, s, taken)              \
                    : launch_waves_slots<WaveTag<n, l, g>, false, true>(A, against, packed, nullptr, s, taken);           \
    return critic ? launch_waves_slots<WaveTag<n, l, g>, true, false>(A, against, packed, critic, s, taken)               \
                  : launch_waves_slots<WaveTag<n, l, g>, false, false>(A, against, packed, nullptr, s, taken);            \
  }
  MPE_TAG_SHAPES(X)
#undef X
  return hipErrorInvalidValue;
}

}  // namespace mpe
