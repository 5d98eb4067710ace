// Status words of a build workspace (internal; not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>

namespace acsc {

// Status words at the head of a build workspace: the Jacobi sweeps used, the
// last sweep's largest off-diagonal ratio and the tolerance (float bits), a
// status (bit 0: the sweep cap was reached above the tolerance; bit 1: the
// Rayleigh-Ritz phase found no stamp of a subspace phase), and the stamp the
// subspace phase leaves for the Rayleigh-Ritz phase, which clears it.
constexpr int kInfoSweeps = 0, kInfoResidual = 1, kInfoTol = 2, kInfoStatus = 3, kInfoStamp = 4, kInfoStall = 5;
constexpr int kStatusNoConv = 1, kStatusNoSubspace = 2, kStatusStalled = 4;
// The stamp a subspace phase leaves for its Rayleigh-Ritz phase: the plain
// one, or the one that also says its fused EMA pass gave up a wait.
constexpr int kSubspaceStamp = 0x5B5D7A11, kSubspaceStalledStamp = 0x5B5D7A13;
// What the fused EMA pass leaves in info[kInfoStall] when one of its bounded
// waits gave up (see sc_pass.h).
constexpr int kEmaStallMark = 0x57A11ED0;

// One thread, near the end of a subspace phase and after its EMA pass: fold
// the stall word into the stamp and clear it for the next phase.
__device__ __forceinline__ void stamp_subspace(int *info)
{
    const bool stalled = info[kInfoStall] == kEmaStallMark;
    info[kInfoStall] = 0;
    info[kInfoStamp] = stalled ? kSubspaceStalledStamp : kSubspaceStamp;
}

}  // namespace acsc
