// Networks small enough that an iteration is bound by its launches and by the
// latency of each: three launches an iteration (small.hip), for one network
// or for a batch of them.
#pragma once

#include "batch_internal.h"

namespace panda {

// Side of the output tiles, and the row-sum slots of C (one per tile of a row).
constexpr int64_t kSmallTile = 32;
inline int64_t small_tiles(int64_t n) { return (n + kSmallTile - 1) / kSmallTile; }
inline int64_t small_h_slots(int64_t Ne, int64_t Na) { return small_tiles(Ne) * small_tiles(Na); }

// Whether a network of this size can take the small kernels (a batch of such
// networks chooses by small_batch), and whether one iterated alone does.
bool small_net(int64_t Ne, int64_t Na);
bool small_run(int64_t Ne, int64_t Na, int32_t precision);

struct SmallRule {
  Rule r;
  int32_t sigma_from_T;
  int32_t packed;
};

// The n networks of `bi` (device descriptors), or the one network `one` where
// bi is null; its W[0] and W[1] are then the old and the new W of the step
// (both the current W outside a step), so that its kernels need not read the
// selector first.  avail: A = T(W, C), the W update and h's partials.  update: h,
// the gates and P's and C's off-diagonals.  finish: both diagonals and R.
// mode kSmallStep: one iteration's; kSmallLoad: update computes only W's norms
// and finish only R, for a state just loaded (both ignore the gates);
// kSmallForce: update regardless of h and the gates (state untouched).
enum SmallMode { kSmallStep = 0, kSmallLoad = 1, kSmallForce = 2 };
// Largest networks of a batch (its grids).
struct SmallDims {
  int64_t Ne, Na;
};
hipError_t launch_small_avail(const BInst* bi, const BInst& one, int n, SmallDims mx,
                              const SmallRule& rule, hipStream_t s);
hipError_t launch_small_update(const BInst* bi, const BInst& one, int n, SmallDims mx,
                               const SmallRule& rule, SmallMode mode, hipStream_t s);
hipError_t launch_small_finish(const BInst* bi, const BInst& one, int n, SmallDims mx,
                               const SmallRule& rule, SmallMode mode, hipStream_t s,
                               DevState* snap = nullptr);  // (one network) pinned copy of the state

}  // namespace panda
