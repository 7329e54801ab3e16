// A maximum over the lanes of a wavefront (DPP).
#pragma once
#include <type_traits>

#include "common.h"

namespace emoe {
namespace {

// The largest of the values that lanes 0 .. LANES-1 hold, GROUP neighbours the same one, in all lanes; 0 where a lane takes no
// part.
template <int LANES, int GROUP>
__device__ __forceinline__ uint32_t max_over_lanes(uint32_t v) {
    auto with = [&](auto ctrl) {
        const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, 0xf, 0xf, true);
        v = v > o ? v : o;
    };
    // row_shr:1, 2, 4, 8: lane 15 of every 16 holds their largest
    if (GROUP < 2) with(std::integral_constant<int, 0x111>{});
    if (GROUP < 4) with(std::integral_constant<int, 0x112>{});
    if (GROUP < 8) with(std::integral_constant<int, 0x114>{});
    if (GROUP < 16) with(std::integral_constant<int, 0x118>{});
    if (LANES > 16 && GROUP < 32) with(std::integral_constant<int, 0x142>{});  // row_bcast:15
    if (LANES > 32 && GROUP < 64) with(std::integral_constant<int, 0x143>{});  // row_bcast:31
    return (uint32_t)__builtin_amdgcn_readlane((int)v, LANES > 32 ? 63 : LANES - 1);
}

}  // namespace
}  // namespace emoe
