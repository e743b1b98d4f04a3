// What the kernels that take one group's list at a time share (pair.hip,
// quad.hip).
#pragma once

#include <type_traits>

#include "common.h"

namespace srf {

// Squared distance from the group's box past which an entry's every pair is
// exactly zero in the FP32 kernels, whose T = 1 - r k / 2 is clamped at 0:
// offsets rounded to FP32 move r by at most 2^-24 times the box size and r
// itself, and r's own arithmetic is good to a few 2^-24.
__device__ __forceinline__ double drop_d2(double far2, double hx, double hy, double hz) {
    const double d = (2.0 * sqrt(far2) + 1e-6 * (hx + hy + hz)) * (1.0 + 4e-6);
    return d * d;
}

__device__ __forceinline__ void lds_order() {
    // one wave: its LDS operations complete in order; this keeps the
    // compiler from moving them across
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Waves per group.  A tree of few groups leaves SIMDs idle, or waiting for
// its longest list, with one wave each; one of many fills the chip either way,
// and waves of one block wait for each other at its end.  Kernel times with 1
// / 4 / 8 waves, us (clustered sets unless said otherwise):
//   groups           force                adjoint
//   240              218 / - / 42         446 / 132 / 89
//   1550             290 / 137 / 137      601 / 283 / 272
//   3050             516 / 234 / 218      1106 / 435 / 435
//   4200 (lattice)   307 / 265 / 281      571 / 503 / 550
//   25000            1468 / 1367 / 1533   2440 / 2340 / 2790
//   51000            2523 / 2476 / 2883   4839 / 4738 / 5809
//   65000 (lattice)  4212 / 4284 / 5074   8120 / 8433 / 10070
//   316000           9841 / 11004 / 14024
constexpr int64_t kOneWaveGroups = 55000;
constexpr int64_t kFourWaveGroups = 3500;

// Calls f with the number of waves per group for ng groups.
template <class F>
void with_waves(int64_t ng, F&& f) {
    if (ng >= kOneWaveGroups) f(std::integral_constant<int, 1>{});
    else if (ng >= kFourWaveGroups) f(std::integral_constant<int, 4>{});
    else f(std::integral_constant<int, 8>{});
}

}  // namespace srf
