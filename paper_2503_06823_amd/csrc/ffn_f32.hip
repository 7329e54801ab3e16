// Expert FFN for fp32 layers (eMoE Section 1: the experts; only slots that received rows are
// touched): grouped GEMM on the fp32 matrix instructions, which multiply and add in full fp32.
//   pass 1: h[r, n] = act(x_perm[r,:] . W1_s[n,:]) (* x_perm[r,:] . W3_s[n,:])
//   pass 2: y_perm[r, n] = h[r,:] . W2_s[n,:]
//
// Bound: the fp32 matrix rate, 256 flop per CU and cycle (the vector units reach half of it without
// packed instructions), as soon as a slot has some tens of rows.
//
// Tile: 32 tokens x 64 weight rows (SwiGLU: 32 of W1 and the same 32 of W3) per workgroup of four
// wavefronts.  fp32 layers are small, and a tile takes the time of a walk along K whatever else is there,
// so tiles are small too: with 32 x 128 the second product of a layer of 1024 tokens, 16 slots,
// d 768, f 3072 (270 tiles) put two walks of 41 us on some CUs and took 95 us.
// Two wavefronts lie side by side along the weight rows and two split every K tile between them (half as
// long a chain of roundings; the halves meet in LDS at the end).  A wavefront holds 2 x 2 blocks of
// v_mfma_f32_16x16x4_f32, for SwiGLU the gate and the up block of the same columns; the second
// 16-token block is skipped when it holds no rows.  The weight rows are the matrix instruction's row
// operand, so a lane ends up with four consecutive output columns of one token.
//
// Data movement: K is walked in tiles of 32 floats (a tile row = one 128-byte line), straight from
// global memory into LDS, 1 KiB per instruction, kStages - 1 tiles ahead.  Chunk c (16 bytes) of row r
// sits at chunk position c ^ ((r >> 1) & 7), which keeps the fragment reads (16 rows x four chunks per
// ds_read_b128) free of bank conflicts.  A fragment read gives a lane four consecutive K elements of its
// row; matrix instruction j multiplies element j of every lane, so that an instruction's four K values
// are 4 apart - the same four in both operands.  Addresses are 64 bit per lane: an fp32 operand may
// exceed what a 32-bit buffer offset reaches.
#include <atomic>
#include <type_traits>

#include "block_sort.h"

namespace emoe {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void;
typedef const __attribute__((address_space(1))) void global_void;

constexpr int BM = 32;              // tokens per tile
constexpr int BR = 64;              // weight rows per tile
constexpr int BK = 32;              // K elements per tile
constexpr int ROW_BYTES = BK * 4;   // 128
constexpr int NW = 4;               // wavefronts: 2 (halves of a K tile) x 2 (along the weight rows)
constexpr int TB = BM / 16;         // 16-token blocks
constexpr int WB = 2;               // 16-row weight blocks per wavefront
constexpr int X_TILE = BM * ROW_BYTES, W_TILE = BR * ROW_BYTES;
constexpr int STAGE_BYTES = X_TILE + W_TILE;  // 12 KiB
constexpr int kStages = 3;          // 36 KiB: four workgroups per CU
constexpr int LX = BM / 8 / NW;     // load instructions per wavefront and K tile: token rows
constexpr int LW = BR / 8 / NW;     // and weight rows
constexpr int LPT = LX + LW;
constexpr int kXcdRun = 16;         // consecutive tiles that go to one XCD
constexpr int kMaxBlocks = 1 << 22; // a grid holds fewer than 2^32 threads
static_assert(BR == 2 * WB * 16, "a wavefront's blocks: gate and up, or two blocks of output columns");

enum Epilogue { kPlain = 0, kSwiglu = 1, kRelu = 2 };

// what K elements past the end of a row are loaded from
__device__ __align__(16) const float kZeros[4] = {0.0f, 0.0f, 0.0f, 0.0f};

// s_waitcnt immediate: vmcnt <= n, all LDS traffic done (vmcnt [3:0] and [15:14], expcnt [6:4], lgkmcnt [11:8])
constexpr int wait_imm(int n) { return (n & 0xf) | ((n >> 4) << 14) | (0x7 << 4) | (0x0 << 8); }

// Workgroup barrier that leaves up to N of this wavefront's global->LDS loads pending (they retire in
// order) and waits for its LDS reads.
template <int N>
__device__ __forceinline__ void barrier_keep_loads() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(wait_imm(N));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// One workgroup per output tile; the launch covers an upper bound of tiles and surplus workgroups exit.
// Tiles are numbered slot by slot, the m-tiles of an n-tile consecutively, and dealt to the XCDs in runs of
// kXcdRun (workgroup ids go round-robin): tiles that share weight rows share an L2, and every XCD has
// tiles of every slot, full and half empty ones.
// Gather: SortingGather if the launch makes the permutation, else RowGather.
template <int EPI, bool KTAIL, class Gather>
__global__ __launch_bounds__(64 * NW, 4) void grouped_gemm_f32(const float* __restrict__ a, Gather gather,
                                                               const int32_t* __restrict__ offsets,
                                                               const float* __restrict__ b0, const float* __restrict__ b1,
                                                               float* __restrict__ c, int S, int N, int K, int n_tiles,
                                                               int XCDS) {
    constexpr int BNO = EPI == kSwiglu ? BR / 2 : BR;  // output columns per tile
    extern __shared__ __align__(16) char lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kh = wave >> 1, wn = wave & 1;

    // ---- this workgroup's tile: lane s holds slot s's rows and the number of its first tile -------------
    BlockSort<NW> sorted;
    constexpr bool sorts = Gather::kSorts;
    if constexpr (sorts) {
        sorted.run(gather.sort, S, reinterpret_cast<int*>(lds));
        if (blockIdx.x == 0) sorted.store_slots(gather.sort, S);
    }
    const int s_begin = sorts ? sorted.begin : lane < S ? offsets[lane] : 0;
    const int s_end = sorts ? sorted.end : lane < S ? offsets[lane + 1] : 0;
    const int s_mtiles = (s_end - s_begin + BM - 1) / BM;
    int incl = s_mtiles * n_tiles;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int up = __shfl_up(incl, off);
        if (lane >= off) incl += up;
    }
    const int first = incl - s_mtiles * n_tiles;
    const int tiles = __builtin_amdgcn_readlane(incl, 63);
    // (one trip, but for launches of more tiles than a grid holds)
    for (int idx = blockIdx.x / XCDS;; idx += gridDim.x / XCDS) {
    const int L = (idx / kXcdRun * XCDS + blockIdx.x % XCDS) * kXcdRun + idx % kXcdRun;
    if (idx / kXcdRun * XCDS * kXcdRun >= tiles) return;
    if (L >= tiles) continue;
    // an empty slot starts where its successor does: the last slot that starts at or before L holds it
    const int slot = __popcll(__ballot(lane < S && first <= L)) - 1;
    const int rem = L - __builtin_amdgcn_readlane(first, slot);
    const int mtiles = __builtin_amdgcn_readlane(s_mtiles, slot);
    const int row0 = __builtin_amdgcn_readlane(s_begin, slot) + (rem % mtiles) * BM;
    const int row_end = __builtin_amdgcn_readlane(s_end, slot);
    const int n0 = (rem / mtiles) * BNO;

    // ---- global -> LDS: instruction (w, i) of an operand fills tile rows (L? w + i) * 8 .. +7; lane l lands in
    //      row l >> 3 of those, chunk position l & 7, and so fetches chunk (l & 7) ^ ((row >> 1) & 7).  Rows past
    //      the slot's end or past N repeat the last one: their results are not stored.
    const int l_row = lane >> 3, l_pos = lane & 7;
    const float* src[LPT];
    int chunk[LPT];
    int* list = reinterpret_cast<int*>(lds + kSortLdsBytes);
    if constexpr (sorts) {
        sorted.list_rows(slot, row0, BM, list);
        if (n0 == 0) sorted.store_rows(gather.sort, slot, row0, BM);
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < LX; ++i) {
        const int tr = (LX * wave + i) * 8 + l_row;
        chunk[i] = l_pos ^ ((tr >> 1) & 7);
        int r = row0 + tr;
        r = r < row_end ? r : row_end - 1;
        // the token's row of x, not a copy of it
        if (gather.perm != nullptr) r = (sorts ? list[r - row0] : gather.perm[r]) / gather.k;
        src[i] = a + (size_t)r * K + chunk[i] * 4;
    }
    if (sorts) __syncthreads();  // the list is read: the stages may be filled
    const float* wsel = (EPI == kSwiglu && wave >= NW / 2) ? b1 : b0;  // wavefronts 2, 3 load the W3 half
#pragma unroll
    for (int i = 0; i < LW; ++i) {
        const int tr = (LW * wave + i) * 8 + l_row;
        chunk[LX + i] = l_pos ^ ((tr >> 1) & 7);
        int n = n0 + (EPI == kSwiglu ? tr % (BR / 2) : tr);
        n = n < N ? n : N - 1;
        src[LX + i] = wsel + ((size_t)slot * N + n) * K + chunk[LX + i] * 4;
    }
    // Every tile walks K from 0: an expert gives the same bits in whichever slot it lies.  Starting the slots at
    // different K tiles, which the bf16 kernels gain from, is worth little here: 70 of 79 layers are level within 3 %, the
    // largest difference is 16 slots of 1 to 8 rows with d 1024, f 4096 (140 / 149 and 170 / 179 us).
    const int k_tiles = (K + BK - 1) / BK;
    auto issue_tile = [&](int stage, int t) {
        const int k0 = t * BK;
        char* base = lds + stage * STAGE_BYTES;
#pragma unroll
        for (int i = 0; i < LPT; ++i) {
            const float* p = src[i] + k0;
            if (KTAIL && k0 + chunk[i] * 4 >= K) p = kZeros;
            char* dst = base + (i < LX ? (LX * wave + i) * 1024 : X_TILE + (LW * wave + i - LX) * 1024);
            __builtin_amdgcn_global_load_lds((global_void*)p, (lds_void*)dst, 16, 0, 0);
        }
    };

    // ---- fragments: lane holds row lane % 16 and, of this wavefront's half kh of a K tile, chunk 4 kh + lane / 16
    const int f_row = lane & 15;
    const int f_sw = (((lane >> 4) + 4 * kh) ^ ((f_row >> 1) & 7)) * 16;
    const int x_off = f_row * ROW_BYTES + f_sw;
    const int w_off = X_TILE + ((EPI == kSwiglu ? wn * 16 : wn * 32) + f_row) * ROW_BYTES + f_sw;
    constexpr int W_STEP = (EPI == kSwiglu ? BR / 2 : 16) * ROW_BYTES;  // from one weight block to the next

    auto tile = [&](auto nb_c) {
        constexpr int NB = decltype(nb_c)::value;  // 16-token blocks that hold rows
        floatx4 acc[WB][NB];
#pragma unroll
        for (int i = 0; i < WB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j) acc[i][j] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
        floatx4 xf[2][NB], wf[2][WB];
        auto load_frags = [&](int buf, int stage) {
            const char* base = lds + stage * STAGE_BYTES;
#pragma unroll
            for (int j = 0; j < NB; ++j) xf[buf][j] = *reinterpret_cast<const floatx4*>(base + x_off + j * 16 * ROW_BYTES);
#pragma unroll
            for (int i = 0; i < WB; ++i) wf[buf][i] = *reinterpret_cast<const floatx4*>(base + w_off + i * W_STEP);
        };
        auto multiply = [&](int buf, int half) {
#pragma unroll
            for (int q = 2 * half; q < 2 * half + 2; ++q)
#pragma unroll
                for (int i = 0; i < WB; ++i)
#pragma unroll
                    for (int j = 0; j < NB; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[buf][i][q], xf[buf][j][q], acc[i][j], 0, 0, 0);
        };
#pragma unroll
        for (int t = 0; t < kStages; ++t)
            if (t < k_tiles) issue_tile(t, t);
        if (k_tiles >= kStages) barrier_keep_loads<(kStages - 1) * LPT>();
        else barrier_keep_loads<0>();
        load_frags(0, 0);
        int stage = 0;
        // The barrier stands inside a K tile's matrix instructions: by then every wavefront holds its fragments of
        // tile t, whose stage takes tile t + kStages, and tile t+1 has landed; the second half of the
        // instructions covers the fragment reads of tile t+1.
        auto k_tile = [&](int buf, int t) {
            const int next = stage + 1 == kStages ? 0 : stage + 1;
            multiply(buf, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (t + kStages <= k_tiles) barrier_keep_loads<(kStages - 2) * LPT>();
            else barrier_keep_loads<0>();
            if (t + kStages < k_tiles) issue_tile(stage, t + kStages);
            load_frags(buf ^ 1, next);  // (past the last tile: whatever the stage holds, not used)
            __builtin_amdgcn_sched_barrier(0);
            multiply(buf, 1);
            __builtin_amdgcn_sched_barrier(0);
            stage = next;
        };
        for (int t = 0; t < k_tiles; t += 2) {
            k_tile(0, t);
            if (t + 1 == k_tiles) break;
            k_tile(1, t + 1);
        }

        // The two halves of K meet in LDS: each wavefront gives its partner one token block and finishes the other.
        // (Nobody reads the stages any more but for the unused fragments, and all loads have landed.)
        barrier_keep_loads<0>();
        floatx4* swap = reinterpret_cast<floatx4*>(lds);  // [wavefront][weight block][lane]
        const int keep = NB == 2 ? kh : 0, give = NB == 2 ? 1 - kh : 0;
        if (NB == 2 || kh == 1) {
#pragma unroll
            for (int i = 0; i < WB; ++i) swap[(wave * WB + i) * 64 + lane] = give == 0 ? acc[i][0] : acc[i][NB - 1];
        }
        barrier_keep_loads<0>();
        if (NB == 2 || kh == 0) {
            // a lane holds token lane % 16 and weight rows 4 (lane / 16) .. +3 of each block
            const int r = row0 + keep * 16 + (lane & 15);
            floatx4 sum[WB];
#pragma unroll
            for (int i = 0; i < WB; ++i)
                sum[i] = (keep == 0 ? acc[i][0] : acc[i][NB - 1]) + swap[((wave ^ 2) * WB + i) * 64 + lane];
            if (r < row_end) {
                const int dr = (EPI == kPlain && gather.out_perm != nullptr) ? gather.out_perm[r] : r;  // combine folded in: the token's row
#pragma unroll
                for (int i = 0; i < (EPI == kSwiglu ? 1 : WB); ++i) {
                    const int n = n0 + (EPI == kSwiglu ? wn * 16 : wn * 32 + i * 16) + (lane >> 4) * 4;
                    if (n >= N) continue;
                    floatx4 v;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        float t = sum[i][q];
                        if (EPI == kSwiglu) t = t / (1.0f + expf(-t)) * sum[WB - 1][q];
                        if (EPI == kRelu) t = fmaxf(t, 0.0f);
                        v[q] = t;
                    }
                    *reinterpret_cast<floatx4*>(c + (size_t)dr * N + n) = v;
                }
            }
        }
        barrier_keep_loads<0>();  // (before another tile's loads)
    };
    static_assert(TB == 2, "written out for one or two token blocks");
    if (row_end - row0 > 16) tile(std::integral_constant<int, 2>{});
    else tile(std::integral_constant<int, 1>{});
    }
}

template <int EPI, bool KTAIL, class Gather>
hipError_t launch_cfg(const float* a, Gather gather, const int32_t* offsets, const float* b0, const float* b1, float* c,
                      long long A, int S, int N, int K, hipStream_t st) {
    constexpr int BNO = EPI == kSwiglu ? BR / 2 : BR;
    constexpr int kLds = kStages * STAGE_BYTES;
    auto kern = grouped_gemm_f32<EPI, KTAIL, Gather>;
    static std::atomic<bool> attr_set{false};  // set once per kernel; setting it twice from two threads is harmless
    if (!attr_set.load(std::memory_order_acquire)) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
        if (e != hipSuccess) return e;
        attr_set.store(true, std::memory_order_release);
    }
    DeviceShape shape;
    hipError_t es = device_shape(&shape);
    if (es != hipSuccess) return es;
    const int n_tiles = (N + BNO - 1) / BNO;
    // every slot adds at most one partial m-tile to the A / BM whole ones
    const long long tiles = (A / BM + (S < A ? S : A)) * n_tiles;
    const long long run = (long long)kXcdRun * shape.xcds;
    const long long rounded = (tiles + run - 1) / run * run, most = kMaxBlocks / run * run;
    const unsigned blocks = (unsigned)(rounded < most ? rounded : most);
    kern<<<blocks, 64 * NW, kLds, st>>>(a, gather, offsets, b0, b1, c, S, N, K, n_tiles, shape.xcds);
    return hipGetLastError();
}

template <int EPI, class Gather>
hipError_t launch_one(const float* a, Gather gather, const int32_t* offsets, const float* b0, const float* b1, float* c,
                      long long A, int S, int N, int K, hipStream_t st) {
    if (K % BK == 0) return launch_cfg<EPI, false>(a, gather, offsets, b0, b1, c, A, S, N, K, st);
    return launch_cfg<EPI, true>(a, gather, offsets, b0, b1, c, A, S, N, K, st);
}

}  // namespace

hipError_t launch_ffn_f32(const emoe_layer_desc& d, const void* x_perm, SortingGather gather, const int32_t* offsets, const void* w1,
                          const void* w3, const void* w2, void* y_perm, void* ws, int passes, hipStream_t st) {
    const long long A = (long long)d.T * d.k;
    float* h = reinterpret_cast<float*>(static_cast<uint8_t*>(ws) + ffn_ws_layout(d).h);
    const float* xp = static_cast<const float*>(x_perm);
    hipError_t e = hipSuccess;
    auto first = [&](auto rows) {
        const float* w1p = static_cast<const float*>(w1);
        if (d.act == EMOE_ACT_SWIGLU)
            return launch_one<kSwiglu>(xp, rows, offsets, w1p, static_cast<const float*>(w3), h, A, d.S, d.d_ff, d.d_model, st);
        return launch_one<kRelu>(xp, rows, offsets, w1p, nullptr, h, A, d.S, d.d_ff, d.d_model, st);
    };
    if (passes & 1) e = gather.sort.A > 0 ? first(gather) : first(RowGather(gather));
    if (e != hipSuccess || !(passes & 2)) return e;
    return launch_one<kPlain>(h, RowGather{nullptr, 1, 0, gather.out_perm}, offsets, static_cast<const float*>(w2), nullptr,
                              static_cast<float*>(y_perm), A, d.S, d.d_model, d.d_ff, st);
}

}  // namespace emoe
