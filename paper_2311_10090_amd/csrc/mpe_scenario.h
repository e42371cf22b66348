// The scenario that a kernel instance runs, as one template parameter: simple spread with N agents (and N landmarks)
// or a predator-prey shape, and the pieces that lane-per-agent kernels of both share.
#pragma once

#include "mpe_tag_device.h"

namespace mpe {

namespace {

template <int N_>
struct SpreadScn {
  static constexpr int N = N_, D = 6 * N_, L = N_;
  static constexpr int LIVE = 4 * N_ + 2;      // leading observation entries that are not always zero
  static constexpr bool kTag = false;
  using Shape = TagShape<2, 1, 1>;             // unused
};
template <int N_, int L_, int G_>
struct TagScn {
  using Shape = TagShape<N_, L_, G_>;
  static constexpr int N = N_, D = Shape::D, L = L_;
  static constexpr int LIVE = D;
  static constexpr bool kTag = true;
};

// Entries 0 .. LIVE - 1 of agent i's observation row into registers (the caller zeroes what lies beyond).
template <typename Scn, int W>
__device__ __forceinline__ void agent_obs(float (&o)[W], int i, float px, float py, float vx, float vy, const float (&qx)[Scn::N],
                                          const float (&qy)[Scn::N], const float (&lx)[Scn::L + 1], const float (&ly)[Scn::L + 1],
                                          const float (&gvx)[Scn::kTag ? Scn::Shape::G : 1], const float (&gvy)[Scn::kTag ? Scn::Shape::G : 1]) {
  constexpr int N = Scn::N;
  if constexpr (Scn::kTag) {
    tag_obs_regs<typename Scn::Shape>(o, i, px, py, vx, vy, qx, qy, lx, ly, gvx, gvy);
  } else {
    o[0] = vx; o[1] = vy; o[2] = px; o[3] = py;
#pragma unroll
    for (int l = 0; l < N; ++l) { o[4 + 2 * l] = lx[l] - px; o[5 + 2 * l] = ly[l] - py; }
    // the k-th OTHER agent is agent k (k < i) or k + 1, ascending
#pragma unroll
    for (int k = 0; k < N - 1; ++k) {
      const bool up = k >= i;
      o[4 + 2 * N + 2 * k] = (up ? qx[k + 1] : qx[k]) - px;
      o[5 + 2 * N + 2 * k] = (up ? qy[k + 1] : qy[k]) - py;
    }
  }
}

}  // namespace

}  // namespace mpe
