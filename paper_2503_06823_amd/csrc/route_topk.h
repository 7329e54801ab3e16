// Resident-restricted top-k of one token by one wavefront, a lane or a group of lanes = expert (eMoE Section 3.2.2), shared by
// all gates: k rounds of a maximum over the lanes (DPP), the lowest lane that holds it wins.  The logits are compared as
// integers of the same order, so that every round has one winner whatever they are; a NaN comes after all numbers.  (With 64
// experts and k = 6 a scan of 32 logits per lane, k times, took some 9 us of a bf16 gate's launch.)  Weights are the softmax
// over the k winners.
#pragma once
#include "wave_max.h"

namespace emoe {
namespace {

// The logit as an integer of the same order, above 0: 1 for a NaN; -0 and +0 are equal.
__device__ __forceinline__ uint32_t logit_order(float logit) {
    const int bits = __float_as_int(logit + 0.0f);
    return logit != logit ? 1u : bits < 0 ? ~(uint32_t)bits : (uint32_t)bits | 0x80000000u;
}

// Lanes e * GROUP .. e * GROUP + GROUP - 1 hold expert e's logit and whether it is resident.  out0: the token's place in the
// outputs.  workload: tokens per expert (the workgroup's in LDS, or the layer's in memory), or nullptr.
template <int EX, int GROUP, class Count>
__device__ __forceinline__ void top_k(float logit, bool resident, int E, int k, size_t out0, int32_t* __restrict__ topk_expert,
                                      float* __restrict__ topk_weight, Count* workload) {
    const int lane = threadIdx.x & 63;
    const uint32_t order = logit_order(logit);
    uint32_t left = resident ? order : 0u;
    int top_v = 0, sel_v = 0, sel_e = 0;  // lane j: the j-th winner
    for (int j = 0; j < k; ++j) {
        const uint32_t best = max_over_lanes<EX * GROUP, GROUP>(left);
        // fewer than k resident experts: precondition broken, stay defined
        const int jl = best ? __builtin_ctzll(__ballot(left == best)) : 0;  // a group's first lane
        const int jv = best ? __builtin_amdgcn_readlane(__float_as_int(logit), jl) : 0;
        left = lane / GROUP == jl / GROUP ? 0u : left;
        if (j == 0) top_v = jv;
        if (lane == j) { sel_v = jv; sel_e = jl / GROUP; }
    }
    const float prob = expf(__int_as_float(sel_v) - __int_as_float(top_v));
    float sum = 0.0f;
    for (int j = 0; j < k; ++j) sum += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(prob), j));
    if (lane < k) {
        topk_expert[out0 + lane] = sel_e;
        topk_weight[out0 + lane] = prob / sum;
    }
    // Workload (Section 3.2.2: the number of tokens an expert receives): the same k rounds over all E
    // experts, resident or not; integer counts, so the accumulated result does not depend on order.
    if (workload != nullptr) {
        left = lane / GROUP < E ? order : 0u;
        bool mine = false;
        for (int j = 0; j < k; ++j) {
            const uint32_t best = max_over_lanes<EX * GROUP, GROUP>(left);
            const int jl = __builtin_ctzll(__ballot(left == best));  // k <= E: best > 0
            left = lane / GROUP == jl / GROUP ? 0u : left;
            mine |= lane == jl;
        }
        if (mine) atomicAdd(&workload[lane / GROUP], (Count)1);
    }
}

}  // namespace
}  // namespace emoe
