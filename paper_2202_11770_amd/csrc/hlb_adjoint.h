// Launchers and device buffers of the adjoint sweep (hlb_adjoint.hip).  Not
// part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "hlb_internal.h"

namespace hlb {

// Partial sums of the objective: each wavefront adds its share to slot
// (wavefront index mod kAdjJSlots), so that no single address takes one
// atomic per wavefront of the grid.
constexpr int64_t kAdjJSlots = 4096;
// Length of AdjBuffers::J: [0] the objective, [8, 8 + kAdjJSlots) the partial
// sums.
constexpr int64_t kAdjJLen = 8 + kAdjJSlots;

// Device buffers of the adjoint sweep (FP64 storage only).
struct AdjBuffers {
  // adjoint of the pre-collision state (tiled, as the state): nu[cur] holds
  // nu_{t+1} before the reverse step t and nu[1 - cur] takes nu_t
  double *nu[2] = {nullptr, nullptr};
  int cur = 0;
  double *J = nullptr;        // [kAdjJLen] objective, partial sums
  double *dA = nullptr;       // [n_iolets][n_steps]
  double *dphi = nullptr;     // [np] porosity derivative per position
  int32_t objective = HLB_OBJ_WSS;
  double *w = nullptr;        // [n_iolets] iolet-flux weights (device)
  int32_t n_io = 0;           // iolets
  double *wq = nullptr;       // [n_iolets] outflow weights of the reverse step in flight
  double *lamX = nullptr;     // [n_iolets] adjoint of the Windkessel outlets' X
};
// Adjoint of the update (t-1 -> t): buffer `src` holds s_{t-1}; b.nu[b.cur]
// holds nu_{t+1} and, in the iolet groups' slots of b.nu[1 - b.cur], mu_t
// (zero before the sweep's first step); on return b.nu[1 - b.cur] holds nu_t
// and the iolet groups' slots of b.nu[b.cur] mu_{t-1}: the caller flips
// b.cur.  Accumulates J's partial sums (if in_window), the iolet table-value
// derivatives into column `step` of dA and the porosity derivatives, and
// forms the outflow weights b.wq (b.lamX must be zero before the sweep's
// first step).
hipError_t launch_adjoint_step(const LaunchCfg &cfg, const Layout &L, const DevPtrs &d, int src, int64_t t,
                               const AdjBuffers &b, int in_window, int64_t n_steps, int64_t step,
                               hipStream_t s);
// J[0] := sum of the partial sums J[8, 8 + kAdjJSlots) (one workgroup).
hipError_t launch_adjoint_objective(double *J, hipStream_t s);

}  // namespace hlb
