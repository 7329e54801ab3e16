// Gate logits and resident-restricted top-k (eMoE Section 1: the gate; Section 3.2.2, last
// paragraph: a token whose expert is not on the GPU goes to its next-best expert that is):
// fp32 inputs with few experts, or with few tokens and long rows, and bf16 inputs when there are few tokens, few
// experts and long rows (a decode step of a Mixtral-shaped layer; up to 16 experts where rows are longer still).  Other fp32
// batches take route_f32.hip, other bf16 batches the matrix-core kernel of route_mfma.hip,
// which puts 16 tokens on a workgroup: with 64 tokens it runs on four CUs, bound by the latency of
// their walk along d_model.
//
// One wavefront (or, when there are few tokens, four) owns one token at a time.  Its 64 lanes
// split the d_model axis (16 bytes per lane per step, so a step reads 1 KiB of the token row
// contiguously); every lane keeps one
// partial sum per expert.  A butterfly reduce-scatter then leaves expert e's complete logit in
// lanes e*(64/EP) .. +64/EP-1: 63 shuffles for 64 experts instead of 64 full reductions.  Top-k: route_topk.h, a group of
// lanes = expert.
// The summation order is fixed by the code, so results are reproducible run to run.
#include <type_traits>

#include "route_topk.h"

namespace emoe {
namespace {

template <typename T> struct Vec;
typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
template <> struct Vec<bf16_t> {
    static constexpr int N = 8;
    typedef uintx4 Raw;
    __device__ static void convert(const uintx4& r, float (&v)[8]) {
        const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[2 * i] = __uint_as_float(w[i] << 16);
            v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        }
    }
};
template <> struct Vec<float> {
    static constexpr int N = 4;
    typedef floatx4 Raw;
    __device__ static void convert(const floatx4& r, float (&v)[4]) {
        v[0] = r.x; v[1] = r.y; v[2] = r.z; v[3] = r.w;
    }
};

// Adds this lane's products of PIECES pieces of the token row (x, x + step) with the gate rows to acc.
// Rows past the last expert repeat that expert's row (their sums are never looked at): without a branch around them
// the loads of all rows are independent.  The loads of GROUP experts go out before any is used: left to itself
// the compiler waits for one expert's pieces after the other, a memory round trip each (gate in HBM, d_model 4096:
// 8 experts 11 -> 6 us, 16 experts 22 -> 10 us).
template <typename T, int EP, int PIECES, int GROUP>
__device__ __forceinline__ void add_pieces(const T* __restrict__ x, const T* __restrict__ w, int step, int d, int E, float (&acc)[EP]) {
    typedef typename Vec<T>::Raw Raw;
    Raw x_raw[PIECES];
#pragma unroll
    for (int h = 0; h < PIECES; ++h) x_raw[h] = *reinterpret_cast<const Raw*>(x + h * step);
#pragma unroll
    for (int e0 = 0; e0 < EP; e0 += GROUP) {
        Raw w_raw[GROUP][PIECES];
#pragma unroll
        for (int e = 0; e < GROUP; ++e)
#pragma unroll
            for (int h = 0; h < PIECES; ++h)
                w_raw[e][h] = *reinterpret_cast<const Raw*>(w + (size_t)(e0 + e < E ? e0 + e : E - 1) * d + h * step);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int h = 0; h < PIECES; ++h) {
            float xv[Vec<T>::N];
            Vec<T>::convert(x_raw[h], xv);
#pragma unroll
            for (int e = 0; e < GROUP; ++e) {
                float wv[Vec<T>::N];
                Vec<T>::convert(w_raw[e][h], wv);
#pragma unroll
                for (int i = 0; i < Vec<T>::N; ++i) acc[e0 + e] = fmaf(xv[i], wv[i], acc[e0 + e]);
            }
        }
    }
}

// EP = number of experts rounded up to a power of two (1..64).
// SPLIT = wavefronts that share one token (1 or 4).  With few tokens (a decode step) one wavefront
// per token would leave most of the chip idle and make each wavefront walk the whole row alone, so
// four wavefronts split the row and add their partial logits through LDS in wavefront order.
// GROUP, PER_CU: experts whose loads go out together, and workgroups that have to fit a CU side by side.
template <typename T, int EP, int SPLIT, int GROUP, int PER_CU>
__global__ __launch_bounds__(256, PER_CU) void route_kernel(const T* __restrict__ x, const T* __restrict__ w_gate,
                                                    const float* __restrict__ bias,
                                                    const int32_t* __restrict__ slot_of_expert,
                                                    int32_t* __restrict__ topk_expert,
                                                    float* __restrict__ topk_weight,
                                                    unsigned long long* __restrict__ expert_tokens, int T_, int d,
                                                    int E, int k) {
    constexpr int VN = Vec<T>::N;
    __shared__ float partial[SPLIT > 1 ? 4 * 64 : 1];
    const int lane = threadIdx.x & 63;
    const int wib = threadIdx.x >> 6;  // wavefront in block
    const int tokens_per_block = 4 / SPLIT;
    const int part = SPLIT > 1 ? wib : 0;  // which share of the row this wavefront sums
    // expert whose logit this lane ends up holding
    const int my_e = lane / (64 / EP);
    const bool resident = my_e < E && slot_of_expert[my_e] >= 0;
    const float my_bias = (bias != nullptr && my_e < E) ? bias[my_e] : 0.0f;

    for (int t0 = blockIdx.x * tokens_per_block; t0 < T_; t0 += gridDim.x * tokens_per_block) {
        const int t = t0 + (SPLIT > 1 ? 0 : wib);
        const bool live = t < T_;  // uniform per wavefront
        float acc[EP];
#pragma unroll
        for (int e = 0; e < EP; ++e) acc[e] = 0.0f;
        if (live) {
            const T* xr = x + (size_t)t * d;
            int c = (part * 64 + lane) * VN;
            const int step = SPLIT * 64 * VN;
            for (; c + step < d; c += 2 * step) add_pieces<T, EP, 2, GROUP>(xr + c, w_gate + c, step, d, E, acc);
            if (c < d) add_pieces<T, EP, 1, GROUP>(xr + c, w_gate + c, step, d, E, acc);
        }
        // butterfly reduce-scatter over the lanes
        int n = EP;
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) {
            if (n > 1) {
                const int half = n / 2;
                const bool upper = (lane & m) != 0;
#pragma unroll
                for (int i = 0; i < half; ++i) {
                    float send = upper ? acc[i] : acc[i + half];
                    float keep = upper ? acc[i + half] : acc[i];
                    acc[i] = keep + __shfl_xor(send, m);
                }
                n = half;
            } else {
                acc[0] += __shfl_xor(acc[0], m);
            }
        }
        float logit = acc[0];
        if (SPLIT > 1) {  // the four shares of the row meet in LDS, added in wavefront order
            partial[wib * 64 + lane] = logit;
            __syncthreads();
            logit = ((partial[lane] + partial[64 + lane]) + partial[128 + lane]) + partial[192 + lane];
            __syncthreads();
            if (wib != 0) continue;
        }
        if (!live) continue;
        logit += my_bias;

        top_k<EP, 64 / EP>(logit, resident, E, k, (size_t)t * k, topk_expert, topk_weight, expert_tokens);
    }
}

constexpr int kWaveRouteTokens = 256;  // bf16, see launch_route()

template <typename T, int EP>
hipError_t launch_ep(const emoe_layer_desc& d, const void* x, const void* w_gate, const float* bias,
                     const int32_t* slot_of_expert, int32_t* topk_expert, float* topk_weight,
                     unsigned long long* expert_tokens, hipStream_t st) {
    const T* xp = static_cast<const T*>(x);
    const T* wg = static_cast<const T*>(w_gate);
    constexpr bool kF32 = std::is_same<T, float>::value;  // bf16: up to kWaveRouteTokens tokens; fp32, EP = 32: up to 2048
    if (!kF32 || d.T <= 2048) {  // fewer than two wavefronts per SIMD otherwise: share each token among four
        int blocks = d.T < 256 * 16 ? d.T : 256 * 16;
        // All experts (16) at a time takes up to 220 registers, which leaves a CU two workgroups.  With more tokens than
        // CUs fp32 rows take four at a time in 128 registers (9 to 16 experts, d_model 2048, 513 to 1000 tokens: 12.0 to 15.1 us
        // against 14.6 to 18.1; d_model 4096, 512 tokens 13.1 against 13.6; 8 experts, d_model 6144, 600 tokens 12.9 against
        // 13.0), and so do 32 experts, whose sums alone are many (64 tokens, d_model 6144: level; 300 tokens: 31.9 us, 16 at a
        // time 49.6).  Four fp32 experts: 72 registers, so that a CU holds seven workgroups (74 made 1537 to 1792 tokens, six to
        // seven workgroups per CU, 1.05 to 1.18 times as slow).
        constexpr int kAll = EP < 16 ? EP : 16;
        constexpr int kPerCu = EP == 32 ? 2 : EP == 4 && kF32 ? 7 : 1;
        auto kern = route_kernel<T, EP, 4, EP == 32 ? 4 : kAll, kPerCu>;
        if constexpr ((EP == 8 || EP == 16) && kF32)
            if (d.T > 256) kern = route_kernel<T, EP, 4, 4, 4>;
        kern<<<blocks, 256, 0, st>>>(xp, wg, bias, slot_of_expert, topk_expert, topk_weight,
                                                       expert_tokens, d.T, d.d_model, d.E, d.k);
    } else if constexpr (kF32 && EP != 32) {
        int blocks = (d.T + 3) / 4;
        if (blocks > 256 * 16) blocks = 256 * 16;
        route_kernel<T, EP, 1, EP < 16 ? EP : 16, 1><<<blocks, 256, 0, st>>>(xp, wg, bias, slot_of_expert, topk_expert, topk_weight,
                                                       expert_tokens, d.T, d.d_model, d.E, d.k);
    }
    return hipGetLastError();
}

template <typename T>
hipError_t launch_t(const emoe_layer_desc& d, const void* x, const void* w_gate, const float* bias,
                    const int32_t* soe, int32_t* te, float* tw, unsigned long long* et, hipStream_t st) {
    if (d.E <= 1) return launch_ep<T, 1>(d, x, w_gate, bias, soe, te, tw, et, st);
    if (d.E <= 2) return launch_ep<T, 2>(d, x, w_gate, bias, soe, te, tw, et, st);
    if (d.E <= 4) return launch_ep<T, 4>(d, x, w_gate, bias, soe, te, tw, et, st);
    if constexpr (std::is_same<T, float>::value) {
        if (d.E > 16 && d.E <= 32 && d.T <= 2048) return launch_ep<T, 32>(d, x, w_gate, bias, soe, te, tw, et, st);
        if (d.E > 16) return launch_ep<T, 64>(d, x, w_gate, bias, soe, te, tw, et, st);
    }
    if (d.E <= 8) return launch_ep<T, 8>(d, x, w_gate, bias, soe, te, tw, et, st);
    return launch_ep<T, 16>(d, x, w_gate, bias, soe, te, tw, et, st);
}

}  // namespace

hipError_t launch_route(const emoe_layer_desc& d, const void* x, const void* w_gate, const float* bias,
                        const int32_t* slot_of_expert, int32_t* topk_expert, float* topk_weight,
                        unsigned long long* expert_tokens, hipStream_t st) {
    if (d.dtype == EMOE_F32) {
        // The matrix kernel reads the gate matrix once per 16 tokens, the wavefront kernel once per token, which is
        // the better one with few experts, or with so few tokens that each has a CU to itself and rows so long that
        // splitting them over more wavefronts counts.  Wavefront / matrix, us a launch in a row of them, k = 2: 8 experts, 1024
        // tokens, d 768 6.0 / 7.1, 8192 tokens 15.2 / 10.8; 4 experts, 8192 tokens, d 2048 19.4 / 17.6.  16 experts, 1024 tokens, d 768
        // 12.3 / 7.4, 64 tokens, d 2048 8.4 / 12.0, 600 tokens, d 2048 13.0 / 12.4, 512 tokens, d 4096 13.0 / 19.6.  32 experts, 64
        // tokens, d 3072 22.0 / 22.8, d 4096 22.9 / 26.7, d 6144 25.8 / 38.9, 300 tokens, d 4096 27.2 / 27.2, d 6144 31.8 / 39.3.  48
        // experts, 64 tokens, d 1536 16.0 / 16.9, d 2048 17.0 / 20.7, d 6144 26.5 / 54, 300 tokens, d 4096 40.7 / 36.5, d 8192 58.6 / 67.7
        // (there the line gives the slower one).  64 experts, 64 tokens, d 768 13.4 / 12.5, d 1536 16.2 / 20.2, 512 tokens, d 2048
        // 35.5 / 25.2, 1024 tokens, d 768 46.3 / 13.0.  At 1000 random gates of more than 16 experts the line takes 1.002 of the
        // better kernel's time in the mean.  With up to 16 experts it does not lie at the crossing: with 9 to 16 and d_model up to
        // 1024 the matrix kernel takes 0.77 to 0.84 of the time with up to 512 tokens already and 0.65 with 513 to 1023, with 5 to 8
        // and d_model up to 1024 0.73 to 1.26 with 2300 to 4096.
        // (A launch of 2^26 tokens would not fit a grid.)
        const int blocks = (d.E + 15) / 16;
        bool matrix = d.E > 8 ? d.T >= 1024 : d.E > 4 && d.T >= 4096;
        if (blocks == 2) matrix = !(d.T <= 512 && d.d_model >= (d.T <= 256 ? 4096 : 5120));
        if (blocks > 2) matrix = !(d.T <= 256 && (long long)d.d_model * blocks >= 6144);
        if (matrix && d.T < (1 << 26))
            return launch_route_f32(d, x, w_gate, bias, slot_of_expert, topk_expert, topk_weight, expert_tokens, st);
        return launch_t<float>(d, x, w_gate, bias, slot_of_expert, topk_expert, topk_weight, expert_tokens, st);
    }
    // bf16: with few tokens and experts a workgroup per token spreads the walk along d_model over more CUs and is
    // better (us a launch in a row of them, wavefront / matrix: 8 experts, d_model 4096, 1 token 5.0 / 6.0, 128 tokens 5.4 /
    // 7.6, 256 tokens 5.6 / 7.6; d_model 8192, 64 tokens 6.7 / 10.9).  With 9 to 16 experts only where rows are long and
    // the tokens not so few (600 gates, matrix / wavefront by d_model up to 4096, 5120, 6144, 7168, 8192, 12000: up to 8 tokens
    // 0.62, 0.71, 0.75, 0.74, 0.79, 0.84; 9 to 16 0.75, 0.91, 0.95, 1.01, 1.00, 1.12; 17 to 64 0.79, 0.97, 1.05, 1.06, 1.11, 1.27; 65 to
    // 256 0.81, 0.97, 1.07, 1.10, 1.19, 1.30).
    const bool few_experts = d.E <= 8 && d.d_model >= 2048;
    const bool long_rows = d.E <= 16 && (d.T > 16 ? d.d_model >= 6144 : d.T > 8 && d.d_model >= 8192);
    if (d.T <= kWaveRouteTokens && (few_experts || long_rows))
        return launch_t<bf16_t>(d, x, w_gate, bias, slot_of_expert, topk_expert, topk_weight, expert_tokens, st);
    return launch_route_bf16(d, x, w_gate, bias, slot_of_expert, topk_expert, topk_weight, expert_tokens, st);
}

}  // namespace emoe
