// Gate logits and resident-restricted top-k for fp32 inputs (eMoE Section 1: the gate; Section 3.2.2, last
// paragraph: a token whose expert is not on the GPU goes to its next-best expert that is), with the logits of
// 16 tokens computed together on the fp32 matrix instructions.
//
// A wavefront per token reads the whole gate matrix for every token, from L2: with 64 experts that is what
// its time goes into (1024 tokens, d_model 768, 64 experts: 66 us; 11 us with this kernel).  Here a workgroup
// owns 16 tokens and every gate row fetched is used for all of them.  Its wavefronts - eight, or sixteen
// with more than 32 experts (15.5 -> 14 us) - split d_model into pieces of 32 floats, loaded straight into
// registers (a lane holds 4 consecutive floats of row lane % 16; a pair of loads covers whole 128-byte
// lines).  The kernel is bound by the latency of that walk, hence few tokens per workgroup and many
// wavefronts.  Partial logits meet in LDS: fp32 accumulation, summation order fixed by the code.
//
// Top-k: a wavefront per token, lane = expert (route_topk.h); before, 16 lanes of one wavefront each scanned their token's
// logits k times (us a launch, d_model 768, 64 experts, 1024 tokens: k = 1 12.7 -> 11.0, k = 8 26.3 -> 12.3; 300
// tokens, d_model 512, 40 experts, k = 6 15.4 -> 7.7; 8192 tokens, d_model 2048, 64 experts, k = 6 72.7 -> 52.1).
#include "route_topk.h"

namespace emoe {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int TOK = 16;    // tokens per workgroup
constexpr int SUMS = 8;    // partial sums per logit that meet in LDS
constexpr int PIECE = 32;  // floats of a row per wavefront and step
constexpr int LDT = TOK + 1;

// EB: blocks of 16 experts.  NW: wavefronts, splitting d_model.
template <int EB, int NW>
__global__ __launch_bounds__(64 * NW) void route_f32_kernel(const float* __restrict__ x, const float* __restrict__ w_gate,
                                                            const float* __restrict__ bias,
                                                            const int32_t* __restrict__ slot_of_expert,
                                                            int32_t* __restrict__ topk_expert,
                                                            float* __restrict__ topk_weight,
                                                            unsigned long long* __restrict__ expert_tokens, int T_, int d,
                                                            int E, int k) {
    constexpr int EX = EB * 16;
    __shared__ float part[SUMS][EX][LDT];
    __shared__ float logit[EX][LDT];
    __shared__ int s_hist[kMaxExperts];  // this workgroup's tokens per expert under ordinary routing
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t0 = blockIdx.x * TOK;
    if (threadIdx.x < kMaxExperts) s_hist[threadIdx.x] = 0;
    const bool resident = lane < E && slot_of_expert[lane] >= 0;  // lane = expert, for the top-k

    // tokens past the last and experts past E repeat the last row; those logits are not looked at
    const int row = lane & 15, at = (lane >> 4) * 4;
    const float* xr = x + (size_t)(t0 + row < T_ ? t0 + row : T_ - 1) * d + at;
    const float* wr[EB];
#pragma unroll
    for (int b = 0; b < EB; ++b) wr[b] = w_gate + (size_t)(16 * b + row < E ? 16 * b + row : E - 1) * d + at;
    floatx4 acc[EB];
#pragma unroll
    for (int b = 0; b < EB; ++b) acc[b] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    struct Piece {
        floatx4 x[2], w[2][EB];
    };
    auto load = [&](Piece& p, int c) {  // floats c .. c + 31 of every row; past d: zeros
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int cc = c + 16 * h;
            const bool ok = cc + at < d;
            p.x[h] = ok ? *reinterpret_cast<const floatx4*>(xr + cc) : floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int b = 0; b < EB; ++b)
                p.w[h][b] = ok ? *reinterpret_cast<const floatx4*>(wr[b] + cc) : floatx4{0.0f, 0.0f, 0.0f, 0.0f};
        }
    };
    // the next piece is on its way while one is multiplied - by the registers, or by the other wavefronts of the SIMD
    constexpr bool AHEAD = NW == SUMS;
    Piece now, then;
    constexpr int STEP = NW * PIECE;
    int c = wave * PIECE;
    if (AHEAD && c < d) load(now, c);
    for (; c < d; c += STEP) {
        if (!AHEAD) load(now, c);
        else if (c + STEP < d) load(then, c + STEP);
        // every instruction starts from zero (four products) and a piece's eight are added as a tree: short chains of
        // roundings, as with a row split over 256 lanes
#pragma unroll
        for (int b = 0; b < EB; ++b) {
            floatx4 p[8];
#pragma unroll
            for (int i = 0; i < 8; ++i)
                p[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(now.w[i >> 2][b][i & 3], now.x[i >> 2][i & 3],
                                                            floatx4{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
            acc[b] += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
        }
        if (AHEAD) now = then;
    }
    // a lane holds token lane % 16 and experts 16 b + 4 (lane / 16) .. +3
    static_assert(NW == SUMS || NW == 2 * SUMS, "the upper wavefronts hand their sums to the lower ones first");
    auto at_part = [&](int b, int q) -> float& { return part[wave % SUMS][16 * b + at + q][row]; };
    if (NW > SUMS) {
        if (wave >= SUMS) {
#pragma unroll
            for (int b = 0; b < EB; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q) at_part(b, q) = acc[b][q];
        }
        __syncthreads();
        if (wave < SUMS) {
#pragma unroll
            for (int b = 0; b < EB; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[b][q] += at_part(b, q);
        }
    }
    if (wave < SUMS) {
#pragma unroll
        for (int b = 0; b < EB; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q) at_part(b, q) = acc[b][q];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < EX * TOK; i += 64 * NW) {
        const int e = i / TOK, t = i % TOK;
        static_assert(SUMS == 8, "written out as a tree");
        const float s = ((part[0][e][t] + part[1][e][t]) + (part[2][e][t] + part[3][e][t])) +
                        ((part[4][e][t] + part[5][e][t]) + (part[6][e][t] + part[7][e][t]));
        logit[e][t] = s + ((bias != nullptr && e < E) ? bias[e] : 0.0f);
    }
    __syncthreads();
#pragma unroll 1
    for (int t = wave; t < TOK && t0 + t < T_; t += NW)
        top_k<EX, 1>(logit[lane < EX ? lane : EX - 1][t], resident, E, k, (size_t)(t0 + t) * k, topk_expert, topk_weight,
                  expert_tokens != nullptr ? s_hist : nullptr);
    if (expert_tokens == nullptr) return;
    __syncthreads();
    if ((int)threadIdx.x < E) {
        const int n = s_hist[threadIdx.x];
        if (n > 0) atomicAdd(&expert_tokens[threadIdx.x], (unsigned long long)n);
    }
}

template <int EB, int NW>
hipError_t launch_eb(const emoe_layer_desc& d, const void* x, const void* w_gate, const float* bias,
                     const int32_t* slot_of_expert, int32_t* topk_expert, float* topk_weight,
                     unsigned long long* expert_tokens, hipStream_t st) {
    route_f32_kernel<EB, NW><<<(unsigned)((d.T + TOK - 1) / TOK), 64 * NW, 0, st>>>(
        static_cast<const float*>(x), static_cast<const float*>(w_gate), bias, slot_of_expert, topk_expert, topk_weight,
        expert_tokens, d.T, d.d_model, d.E, d.k);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_route_f32(const emoe_layer_desc& d, const void* x, const void* w_gate, const float* bias,
                            const int32_t* slot_of_expert, int32_t* topk_expert, float* topk_weight,
                            unsigned long long* expert_tokens, hipStream_t st) {
    switch ((d.E + 15) / 16) {
        case 1: return launch_eb<1, 8>(d, x, w_gate, bias, slot_of_expert, topk_expert, topk_weight, expert_tokens, st);
        case 2: return launch_eb<2, 8>(d, x, w_gate, bias, slot_of_expert, topk_expert, topk_weight, expert_tokens, st);
        case 3: return launch_eb<3, 16>(d, x, w_gate, bias, slot_of_expert, topk_expert, topk_weight, expert_tokens, st);
        default: return launch_eb<4, 16>(d, x, w_gate, bias, slot_of_expert, topk_expert, topk_weight, expert_tokens, st);
    }
}

}  // namespace emoe
