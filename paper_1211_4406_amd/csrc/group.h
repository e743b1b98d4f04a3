// What the kernels that take one group's list at a time share (pair.hip,
// quad.hip).
#pragma once

#include <type_traits>

#include "common.h"
#include "waves.h"

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

// Calls f with the number of waves per group for these lists.
template <class F>
void with_waves(const Lists& l, double reach, F&& f) {
    const int w = waves_per_group(l.n_groups, l.n_entries, l.interactions, reach);
    if (w == 1) f(std::integral_constant<int, 1>{});
    else if (w == 4) f(std::integral_constant<int, 4>{});
    else f(std::integral_constant<int, 8>{});
}

}  // namespace srf
