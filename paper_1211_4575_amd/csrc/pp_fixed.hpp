// Scale of the split form's fixed-point current.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "../../include/pp.h"
#include "pp_device.hpp"

struct pp_run;

namespace pp {

struct FixedScale {
    const int32_t* tile_max;  // largest tile population per species slot (device)
    int e0;                   // host part of the exponent
};

FixedScale gpd32_scale(const pp_run* r);

// 2^e with e = e0 - ceil(log2(N)), N the sum over species of the largest particle count of
// any tile: then |one contribution| <= 2^(50 - ceil log2 N) and |a node's LDS sum| <= 2^50.
// Eight loads of one line: every kernel that needs the scale works it out itself.
__device__ __forceinline__ double fixed_scale(const FixedScale& F) {
    long long nb = 0;
#pragma unroll
    for (int s = 0; s < PP_MAX_SPECIES; ++s) nb += gl(F.tile_max)[s];
    const int e = __builtin_amdgcn_readfirstlane(F.e0 - (nb > 1 ? 64 - __clzll(nb - 1) : 0));  // uniform
    if (e >= -1022 && e <= 1023) return __longlong_as_double((long long)(e + 1023) << 52);
    return ldexp(1.0, e);
}

}  // namespace pp
