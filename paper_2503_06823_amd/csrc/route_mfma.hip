// Gate logits and resident-restricted top-k for bf16 inputs (eMoE Section 1: the gate; Section
// 3.2.2, last paragraph: a token whose expert is not on the GPU goes to its next-best expert that
// is), with the logits of 16 or 32 tokens computed together on the matrix cores.
//
// A wavefront per token re-reads the whole gate matrix per token; here a workgroup owns 16 tokens (32
// when 16 would give more workgroups than the chip has CUs), and every gate row fetched is used for
// all of them: v_mfma_f32_16x16x32_bf16 with gate rows on the row and token rows on the column
// operand.  What bounds it is the latency of the walk along d_model and the rate at which a CU moves gate rows into LDS.
// Four to sixteen wavefronts share the walk in pieces of 64 elements.  A piece (128 bytes, one line, of every token and gate
// row) goes from global memory straight into LDS with buffer_load_dwordx4 ... lds, 1 KiB of whole lines per
// instruction (a register load in the operand's layout puts 16 rows side by side in its lanes and is bound by the L1's
// tag rate: 100 tokens, d_model 4096, 64 experts 23 us, 13 with LDS), into a ring of the wavefront's own: a
// wavefront waits for nobody, there is no barrier in the walk.  All of LDS is ring.
// In LDS the 16-byte chunk c of row r sits at chunk position c ^ ((r >> 1) & 7), which makes the fragment reads (16 rows
// x one chunk) bank-conflict free.
// Measured (us a launch, x from HBM; before, with 32 tokens, four wavefronts and a barrier per tile): 1024 tokens, d_model
// 4096, 8 experts 11.8 -> 5.9; 4096 of them 15.1 -> 10.1 (3.4 TB/s of x); 512 tokens, d_model 2048, 64 experts, k = 6 16.5 ->
// 7.6; 8192 of them 21.2 -> 15.5; 64 tokens, d_model 768, 64 experts 7.0 -> 4.2; one token 13.4 -> 4.8 (d_model 1024).
//
// The partial sums of a logit meet in LDS and are added as a tree: fp32 accumulation, summation
// order fixed by the code.
//
// Top-k: a wavefront per token, lane = expert (route_topk.h).
#include <atomic>

#include "route_topk.h"

namespace emoe {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

typedef __attribute__((address_space(3))) void lds_void;

constexpr int NW = 16;                    // wavefronts: all of them for the top-k, the first NL for the walk along d_model
constexpr int PIECE = 64;                 // elements of a row per wavefront and step
constexpr int ROW_BYTES = PIECE * 2;      // 128
constexpr int kLdsBytes = 160 * 1024;     // of one CU
constexpr unsigned kRotation = 21;        // rotation of the walk per workgroup

// s_waitcnt immediate: vmcnt <= n and all LDS traffic done (vmcnt[3:0] | [15:14], expcnt [6:4], lgkmcnt [11:8])
constexpr int wait_imm(int n) { return (n & 0xf) | ((n >> 4) << 14) | (0x7 << 4) | (0x0 << 8); }
template <int N>
__device__ __forceinline__ void wait_loads() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(wait_imm(N));
    asm volatile("" ::: "memory");
}

// What follows from the blocks of 16 experts and 16 tokens: the wavefronts that walk, the pieces in flight in each.
template <int EB, int TB>
struct Shape {
    static constexpr int EX = 16 * EB, TOK = 16 * TB;
    static constexpr int PIECE_BYTES = (EX + TOK) * ROW_BYTES;
    static constexpr int LOADS = PIECE_BYTES / 1024;                              // load instructions per piece
    static constexpr int NL = 16 * 2 * PIECE_BYTES <= kLdsBytes ? 16 : 8 * 2 * PIECE_BYTES <= kLdsBytes ? 8 : 4;
    static constexpr int FIT = kLdsBytes / (NL * PIECE_BYTES), DEPTH = FIT < 4 ? FIT : 4;
    static constexpr int LDE = EX + 4;  // a token's logits, padded: 16-byte stores of 16 tokens spread over the banks
    static constexpr int SUM_BYTES = NL * TOK * LDE * (int)sizeof(float);         // reuses the rings, and so does
    static constexpr int LDS = NL * DEPTH * PIECE_BYTES;                          // the histogram behind it
    static_assert(SUM_BYTES + kMaxExperts * (int)sizeof(int) <= LDS && LDS <= kLdsBytes, "LDS of one CU");
    static_assert((DEPTH - 1) * LOADS < 64, "vmcnt counts at most 63 loads");
};

// EB: blocks of 16 experts.  TB: blocks of 16 tokens.
template <int EB, int TB>
__global__ __launch_bounds__(64 * NW) void route_mfma_kernel(const bf16_t* __restrict__ x,
                                                             const bf16_t* __restrict__ w_gate,
                                                             const float* __restrict__ bias,
                                                             const int32_t* __restrict__ slot_of_expert,
                                                             int32_t* __restrict__ topk_expert,
                                                             float* __restrict__ topk_weight,
                                                             unsigned long long* __restrict__ expert_tokens, int T_,
                                                             int K, int E, int k) {
    typedef Shape<EB, TB> Sh;
    constexpr int EX = Sh::EX, TOK = Sh::TOK, NL = Sh::NL, LOADS = Sh::LOADS, DEPTH = Sh::DEPTH, LDE = Sh::LDE;
    extern __shared__ __align__(16) char lds[];
    float* part = reinterpret_cast<float*>(lds);                   // [wavefront][token][LDE], once the rings are read
    int* s_hist = reinterpret_cast<int*>(lds + Sh::SUM_BYTES);     // this workgroup's tokens per expert under ordinary routing
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t0 = blockIdx.x * TOK;
    // lane = expert, for the second half
    const float lane_bias = (bias != nullptr && lane < E) ? bias[lane] : 0.0f;
    const bool resident = lane < E && slot_of_expert[lane] >= 0;

    // with up to 16 experts the halves of a piece have sums of their own: chains of roundings half as long
    constexpr int HALVES = EB == 1 ? 2 : 1;
    floatx4 acc[HALVES][EB][TB];
#pragma unroll
    for (int h = 0; h < HALVES; ++h)
#pragma unroll
        for (int b = 0; b < EB; ++b)
#pragma unroll
            for (int j = 0; j < TB; ++j) acc[h][b][j] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    if (wave < NL) {
        // Load instruction i fills rows 8 i .. 8 i + 7 of a piece, gate rows first; lane l lands in row l / 8 of those, chunk
        // position l % 8.  Rows past the last token or expert and chunks past K are addressed out of range: zeros.
        const int l_row = lane >> 3, l_pos = lane & 7;
        const uint32_t x_bytes = (uint32_t)T_ * (uint32_t)K * 2u, w_bytes = (uint32_t)E * (uint32_t)K * 2u;
        const __amdgpu_buffer_rsrc_t x_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(x), 0, (int)x_bytes, 0x00020000);
        const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(w_gate), 0, (int)w_bytes, 0x00020000);
        uint32_t voff[LOADS];
        int chunk[2];  // of load i: by its parity
#pragma unroll
        for (int i = 0; i < 2; ++i) chunk[i] = l_pos ^ (((8 * i + l_row) >> 1) & 7);
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const int r = 8 * i + l_row;
            if (8 * i < EX) voff[i] = r < E ? ((uint32_t)r * (uint32_t)K + chunk[i & 1] * 8) * 2u : w_bytes;
            else voff[i] = t0 + r - EX < T_ ? ((uint32_t)(t0 + r - EX) * (uint32_t)K + chunk[i & 1] * 8) * 2u : x_bytes;
        }
        const int pieces = (K + PIECE - 1) / PIECE;
        // Workgroups start at different pieces of K: token rows are a power-of-two-ish stride apart, so workgroups that
        // march through K in step would all pull from the same few HBM channels.  The order is fixed per workgroup.
        const int rot = (int)((blockIdx.x * kRotation) % (unsigned)pieces);
        char* ring = lds + wave * DEPTH * Sh::PIECE_BYTES;
        auto issue = [&](int slot, int p) {  // past the last piece: out of range too, so that every wait counts the same
            int pp = p + rot;
            pp = pp >= pieces ? pp - pieces : pp;
            const int k0 = p < pieces ? pp * PIECE : K;
            const bool out[2] = {k0 + chunk[0] * 8 >= K, k0 + chunk[1] * 8 >= K};
#pragma unroll
            for (int i = 0; i < LOADS; ++i) {
                const bool gate = 8 * i < EX;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(gate ? w_rsrc : x_rsrc,
                                                         (lds_void*)(ring + slot * Sh::PIECE_BYTES + i * 1024), 16,
                                                         (int)(out[i & 1] ? (gate ? w_bytes : x_bytes) : voff[i]),
                                                         p < pieces ? k0 * 2 : 0, 0, 0);
            }
        };
        // fragments: lane holds row lane % 16 and, of half h of the piece, chunk 4 h + lane / 16
        const int row = lane & 15, sw = (row >> 1) & 7;
        const int f_off = row * ROW_BYTES;
#pragma unroll
        for (int s = 0; s < DEPTH - 1; ++s) issue(s, wave + s * NL);
        int slot = 0;
        for (int p = wave; p < pieces; p += NL) {
            const int ahead = slot == 0 ? DEPTH - 1 : slot - 1;  // read in the last trip: its LDS reads are done (below)
            issue(ahead, p + (DEPTH - 1) * NL);
            wait_loads<(DEPTH - 1) * LOADS>();
            const char* at = ring + slot * Sh::PIECE_BYTES + f_off;
            bf16x8 wf[2][EB], xf[2][TB];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int c = ((4 * h + (lane >> 4)) ^ sw) * 16;
#pragma unroll
                for (int b = 0; b < EB; ++b) wf[h][b] = *reinterpret_cast<const bf16x8*>(at + b * 16 * ROW_BYTES + c);
#pragma unroll
                for (int j = 0; j < TB; ++j) xf[h][j] = *reinterpret_cast<const bf16x8*>(at + (EX + j * 16) * ROW_BYTES + c);
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int b = 0; b < EB; ++b)
#pragma unroll
                    for (int j = 0; j < TB; ++j)
                        acc[h % HALVES][b][j] =
                            __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[h][b], xf[h][j], acc[h % HALVES][b][j], 0, 0, 0);
            wait_loads<63>();  // the fragments are in registers: the next trip's loads may overwrite this piece
            slot = slot + 1 == DEPTH ? 0 : slot + 1;
        }
        wait_loads<0>();  // surplus loads have landed too
    }
    __syncthreads();  // the rings are read: the partial sums may overwrite them
    if (wave < NL) {
        // a lane holds token lane % 16 and experts 16 b + 4 (lane / 16) .. +3
#pragma unroll
        for (int j = 0; j < TB; ++j)
#pragma unroll
            for (int b = 0; b < EB; ++b)
                *reinterpret_cast<floatx4*>(part + (size_t)(wave * TOK + 16 * j + (lane & 15)) * LDE + 16 * b + (lane >> 4) * 4) =
                    HALVES == 2 ? acc[0][b][j] + acc[HALVES - 1][b][j] : acc[0][b][j];
    }
    if (wave == NW - 1) s_hist[lane] = 0;
    __syncthreads();

#pragma unroll 1
    for (int tt = wave; tt < TOK && t0 + tt < T_; tt += NW) {
        float s[NL];
        const int e = lane < EX ? lane : EX - 1;
#pragma unroll
        for (int w = 0; w < NL; ++w) s[w] = part[(size_t)(w * TOK + tt) * LDE + e];
#pragma unroll
        for (int n = NL / 2; n > 0; n /= 2)
#pragma unroll
            for (int w = 0; w < n; ++w) s[w] += s[w + n];
        const float logit = s[0] + lane_bias;
        top_k<EX, 1>(logit, resident, E, k, (size_t)(t0 + tt) * k, topk_expert, topk_weight, expert_tokens != nullptr ? s_hist : nullptr);
    }
    if (expert_tokens == nullptr) return;
    __syncthreads();
    if ((int)threadIdx.x < E) {
        const int n = s_hist[threadIdx.x];
        if (n > 0) atomicAdd(&expert_tokens[threadIdx.x], (unsigned long long)n);
    }
}

template <int EB, int TB>
hipError_t launch_tb(const emoe_layer_desc& d, const bf16_t* x, const bf16_t* wg, const float* bias,
                     const int32_t* slot_of_expert, int32_t* topk_expert, float* topk_weight,
                     unsigned long long* expert_tokens, hipStream_t st) {
    constexpr int kLds = Shape<EB, TB>::LDS, TOK = Shape<EB, TB>::TOK;
    auto kern = route_mfma_kernel<EB, TB>;
    static std::atomic<bool> attr_set{false};  // set once per kernel; setting it twice from two threads is harmless
    if (!attr_set.load(std::memory_order_acquire)) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
        if (e != hipSuccess) return e;
        attr_set.store(true, std::memory_order_release);
    }
    kern<<<(unsigned)(((long long)d.T + TOK - 1) / TOK), 64 * NW, kLds, st>>>(x, wg, bias, slot_of_expert, topk_expert, topk_weight,
                                                                             expert_tokens, d.T, d.d_model, d.E, d.k);
    return hipGetLastError();
}

template <int EB>
hipError_t launch_eb(const emoe_layer_desc& d, const bf16_t* x, const bf16_t* wg, const float* bias,
                     const int32_t* slot_of_expert, int32_t* topk_expert, float* topk_weight,
                     unsigned long long* expert_tokens, hipStream_t st) {
    DeviceShape shape;
    hipError_t e = device_shape(&shape);
    if (e != hipSuccess) return e;
    // 32 tokens per workgroup fetch the gate rows half as often; 16 fill the chip with fewer tokens and have
    // half the top-k to do (16 against 32: 4200 tokens, d_model 2048, 64 experts 14.4 / 10.7 us, 8192 of d_model 1024, 16
    // experts 8.4 / 6.8; at 4096 tokens 32 would leave half the CUs idle).
    if (d.T <= 16 * shape.cus)
        return launch_tb<EB, 1>(d, x, wg, bias, slot_of_expert, topk_expert, topk_weight, expert_tokens, st);
    return launch_tb<EB, 2>(d, x, wg, bias, slot_of_expert, topk_expert, topk_weight, expert_tokens, st);
}

}  // namespace

hipError_t launch_route_bf16(const emoe_layer_desc& d, const void* x, const void* w_gate, const float* bias,
                             const int32_t* slot_of_expert, int32_t* topk_expert, float* topk_weight,
                             unsigned long long* expert_tokens, hipStream_t st) {
    const bf16_t* xp = static_cast<const bf16_t*>(x);
    const bf16_t* wg = static_cast<const bf16_t*>(w_gate);
    switch ((d.E + 15) / 16) {
        case 1: return launch_eb<1>(d, xp, wg, bias, slot_of_expert, topk_expert, topk_weight, expert_tokens, st);
        case 2: return launch_eb<2>(d, xp, wg, bias, slot_of_expert, topk_expert, topk_weight, expert_tokens, st);
        case 3: return launch_eb<3>(d, xp, wg, bias, slot_of_expert, topk_expert, topk_weight, expert_tokens, st);
        default: return launch_eb<4>(d, xp, wg, bias, slot_of_expert, topk_expert, topk_weight, expert_tokens, st);
    }
}

}  // namespace emoe
