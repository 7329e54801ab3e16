// Expert FFN for bf16 layers of at most 16 tokens (a decode step of a few users; eMoE Section 5.1: fewer experts means
// fewer global-memory reads): no more slots than assignments receive rows, each at most 16 (a token's k experts are
// different; a caller's own assignments may put more into a slot, 16 per pass over its weights), and the cost is reading those
// slots' weights from HBM once, or, for small layers, the latency of one walk along K.
//
// A workgroup owns 32 weight rows of one slot (SwiGLU: 16 rows of W1 and the same 16 of W3), 16 where 32 would leave
// half the CUs without any, or 64 where the walks are short and the workgroups many.  Its wavefronts share K in pieces
// of 64 elements: a piece (128 bytes, one line, of every weight row and of 16 token rows) goes from global memory straight into LDS with buffer_load_dwordx4 ... lds, into a ring of
// the wavefront's own.  A wavefront waits for its own loads only, so there is no barrier in the walk and short walks
// have all their loads on the way at once.  Sixteen token rows instead of 32 leave LDS for weights: 96 KiB of them
// in flight per CU, in two workgroups of four wavefronts or, where there are no more workgroups than CUs, in one of eight.
// Measured (us, weights from HBM, first + second product; before, 32 token rows, a barrier per tile of 128): one token, d 4096,
// f 14336, two slots 83 + 54 -> 71 + 39 (6.1 TB/s); 8 tokens, 8 slots 282 + 139 -> 260 + 139; one token, d 2048, f 8192, two of
// 16 slots 26 + 31 -> 24 + 16; d 512, f 2048, top-1, ReLU 4.4 + 6.4 -> 4.1 + 5.2.
//
// In LDS the 16-byte chunk c of row r sits at chunk position c ^ ((r >> 1) & 7): the fragment reads of
// v_mfma_f32_16x16x32_bf16 (16 rows x one chunk) are bank-conflict free.  Weight rows are the row operand, tokens the column
// operand.  The wavefronts' sums meet in LDS and are added in wavefront order.
//
// The launch covers as many slots as can hold rows, at most one per assignment; a workgroup finds its slot as the n-th that does.
#include <atomic>

#include "block_sort.h"

namespace emoe {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void;

enum Epilogue { kPlain = 0, kSwiglu = 1, kRelu = 2 };

constexpr int TOK = 16;               // token rows per pass
constexpr int PIECE = 64;             // elements of a row per wavefront and step
constexpr int ROW_BYTES = PIECE * 2;  // 128
constexpr unsigned kRotation = 21;    // rotation of the walk per workgroup
constexpr int kLongK = 2048, kShortK = 512;  // see launch_one()
constexpr int kStreamOnce = 2;        // non-temporal hint of the weight loads

constexpr int wait_imm(int n) { return (n & 0xf) | ((n >> 4) << 14) | (0x7 << 4) | (0x0 << 8); }
// At most N of this wavefront's global->LDS loads pending (they retire in order), its LDS reads done.
template <int N>
__device__ __forceinline__ void wait_loads() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(wait_imm(N));
    asm volatile("" ::: "memory");
}

template <int WR, int WAVES>
struct Shape {
    static constexpr int PIECE_BYTES = (WR + TOK) * ROW_BYTES;
    static constexpr int LOADS = PIECE_BYTES / 1024;
    static constexpr int FIT = (WAVES == 8 ? 160 : 80) * 1024 / (WAVES * PIECE_BYTES), DEPTH = FIT < 5 ? FIT : 5;
    static constexpr int LDS = WAVES * DEPTH * PIECE_BYTES;
    static_assert(DEPTH >= 2 && (DEPTH - 1) * LOADS < 64, "vmcnt counts at most 63 loads");
    static_assert(WAVES * (WR / 16) * 64 * 16 <= LDS, "the sums reuse the rings");
};

// Gather: SortingGather if the launch makes the permutation, else RowGather.
template <int EPI, int WR, int WAVES, bool ONCE, class Gather>
__global__ __launch_bounds__(64 * WAVES) void few_gemm_bf16(const bf16_t* __restrict__ a, Gather gather,
                                                           const int32_t* __restrict__ offsets,
                                                           const bf16_t* __restrict__ b0, const bf16_t* __restrict__ b1,
                                                           bf16_t* __restrict__ c, int S, int N, int K, int n_units) {
    typedef Shape<WR, WAVES> Sh;
    constexpr int NBLK = WR / 16, LOADS = Sh::LOADS, DEPTH = Sh::DEPTH;
    constexpr int BNO = EPI == kSwiglu ? WR / 2 : WR;  // output columns
    static_assert(EPI != kSwiglu || WR >= 32, "as many blocks of gate rows as of up rows");
    constexpr int OUT_BLK = BNO / 16;  // output column blocks
    extern __shared__ __align__(16) char lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    BlockSort<WAVES> sorted;
    constexpr bool sorts = Gather::kSorts;
    if constexpr (sorts) {
        sorted.run(gather.sort, S, reinterpret_cast<int*>(lds));
        if (blockIdx.x == 0) sorted.store_slots(gather.sort, S);
    }
    const int s_begin = sorts ? sorted.begin : lane < S ? offsets[lane] : 0;
    const int s_end = sorts ? sorted.end : lane < S ? offsets[lane + 1] : 0;
    unsigned long long used = __ballot(s_end > s_begin);
    int nth = blockIdx.x / n_units;
    if (nth >= __popcll(used)) return;
    for (; nth > 0; --nth) used &= used - 1;
    const int slot = __builtin_ctzll(used);
    const int row0 = __builtin_amdgcn_readlane(s_begin, slot), row_end = __builtin_amdgcn_readlane(s_end, slot);
    const int rows_total = __builtin_amdgcn_readlane(s_end, S - 1);
    const int n0 = (blockIdx.x % n_units) * BNO;

    // Load instruction i fills rows 8 i .. 8 i + 7 of a piece, weight rows first; lane l lands in row l / 8 of those, chunk
    // position l % 8.  Rows past the matrix or the slot and chunks past K are addressed out of range: zeros, no traffic.
    const int l_row = lane >> 3, l_pos = lane & 7;
    const uint32_t a_bytes = (uint32_t)(gather.perm != nullptr ? gather.rows : rows_total) * (uint32_t)K * 2u;
    const uint32_t b_bytes = (uint32_t)N * (uint32_t)K * 2u;
    const __amdgpu_buffer_rsrc_t a_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a), 0, (int)a_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t b0_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(b0 + (size_t)slot * N * K), 0,
                                                                            (int)b_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t b1_rsrc = EPI != kSwiglu ? b0_rsrc : __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t*>(b1 + (size_t)slot * N * K), 0, (int)b_bytes, 0x00020000);
    int chunk[2];  // of load i: by its parity
#pragma unroll
    for (int i = 0; i < 2; ++i) chunk[i] = l_pos ^ (((8 * i + l_row) >> 1) & 7);
    uint32_t voff[LOADS];
#pragma unroll
    for (int i = 0; i < WR / 8; ++i) {
        const int tr = 8 * i + l_row;
        const int n = n0 + (EPI == kSwiglu ? tr % BNO : tr);
        voff[i] = n < N ? ((uint32_t)n * (uint32_t)K + chunk[i & 1] * 8) * 2u : b_bytes;
    }
    const int pieces = (K + PIECE - 1) / PIECE;
    // Workgroups start at different pieces of K: rows are a power-of-two-ish stride apart, and workgroups that march
    // through K in step would all pull from the same few HBM channels.  The order is fixed per workgroup.
    const int rot = (int)((blockIdx.x * kRotation) % (unsigned)pieces);
    char* ring = lds + wave * DEPTH * Sh::PIECE_BYTES;
    const int f_off = (lane & 15) * ROW_BYTES, f_sw = ((lane & 15) >> 1) & 7;

    for (int tok0 = row0; tok0 < row_end; tok0 += TOK) {
        int* list = reinterpret_cast<int*>(lds + kSortLdsBytes);
        if constexpr (sorts) {
            sorted.list_rows(slot, tok0, TOK, list);
            if (n0 == 0) sorted.store_rows(gather.sort, slot, tok0, TOK);
            __syncthreads();
        }
#pragma unroll
        for (int i = WR / 8; i < LOADS; ++i) {
            int r = tok0 + 8 * (i - WR / 8) + l_row;
            const bool past = r >= row_end;
            r = past ? row_end - 1 : r;
            // the token's row of x, not a copy of it
            if (gather.perm != nullptr) r = (sorts ? list[r - tok0] : gather.perm[r]) / gather.k;
            voff[i] = past ? a_bytes : ((uint32_t)r * (uint32_t)K + chunk[i & 1] * 8) * 2u;
        }
        if (sorts) __syncthreads();  // the list is read: the rings may be filled
        auto issue = [&](int at, int p) {  // past the last piece: out of range too, so that every wait counts the same
            int pp = p + rot;
            pp = pp >= pieces ? pp - pieces : pp;
            const int k0 = p < pieces ? pp * PIECE : 0;
            const bool out[2] = {p >= pieces || k0 + chunk[0] * 8 >= K, p >= pieces || k0 + chunk[1] * 8 >= K};
#pragma unroll
            for (int i = 0; i < LOADS; ++i) {
                lds_void* dst = (lds_void*)(ring + at * Sh::PIECE_BYTES + i * 1024);
                if (i < WR / 8)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(EPI == kSwiglu && i >= WR / 16 ? b1_rsrc : b0_rsrc, dst, 16,
                                                             (int)(out[i & 1] ? b_bytes : voff[i]), k0 * 2, 0, ONCE ? kStreamOnce : 0);
                else
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rsrc, dst, 16, (int)(out[i & 1] ? a_bytes : voff[i]), k0 * 2, 0, 0);
            }
        };
        floatx4 acc[NBLK];
#pragma unroll
        for (int b = 0; b < NBLK; ++b) acc[b] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int s = 0; s < DEPTH - 1; ++s) issue(s, wave + s * WAVES);
        int at = 0;
        for (int p = wave; p < pieces; p += WAVES) {
            issue(at == 0 ? DEPTH - 1 : at - 1, p + (DEPTH - 1) * WAVES);  // read in the last trip: its LDS reads are done (below)
            wait_loads<(DEPTH - 1) * LOADS>();
            const char* base = ring + at * Sh::PIECE_BYTES + f_off;
            bf16x8 wf[2][NBLK], xf[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int cc = ((4 * h + (lane >> 4)) ^ f_sw) * 16;
#pragma unroll
                for (int b = 0; b < NBLK; ++b) wf[h][b] = *reinterpret_cast<const bf16x8*>(base + b * 16 * ROW_BYTES + cc);
                xf[h] = *reinterpret_cast<const bf16x8*>(base + WR * ROW_BYTES + cc);
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int b = 0; b < NBLK; ++b) acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[h][b], xf[h], acc[b], 0, 0, 0);
            wait_loads<63>();  // the fragments are in registers: the next trip's loads may overwrite this piece
            at = at + 1 == DEPTH ? 0 : at + 1;
        }
        wait_loads<0>();  // surplus loads have landed too
        __syncthreads();  // the rings are read: the sums may overwrite them
        floatx4* part = reinterpret_cast<floatx4*>(lds);  // [block][wavefront][lane]
#pragma unroll
        for (int b = 0; b < NBLK; ++b) part[(b * WAVES + wave) * 64 + lane] = acc[b];
        __syncthreads();
        // wavefront b: output block b; a lane holds token lane % 16, columns 4 (lane / 16) .. +3
        if (wave < OUT_BLK) {
            auto sum = [&](int b) {
                floatx4 v = part[b * WAVES * 64 + lane];
#pragma unroll
                for (int w = 1; w < WAVES; ++w) v += part[(b * WAVES + w) * 64 + lane];
                return v;
            };
            floatx4 v = sum(wave);
            if (EPI == kSwiglu) {
                const floatx4 up = sum(wave + OUT_BLK);
#pragma unroll
                for (int q = 0; q < 4; ++q) v[q] = v[q] / (1.0f + __expf(-v[q])) * up[q];
            }
            const int r = tok0 + (lane & 15), n = n0 + wave * 16 + (lane >> 4) * 4;
            if (r < row_end && n < N) {
                if (EPI == kRelu) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) v[q] = fmaxf(v[q], 0.0f);
                }
                const int dr = (EPI == kPlain && gather.out_perm != nullptr) ? gather.out_perm[r] : r;  // combine folded in
                *reinterpret_cast<bf16x4*>(c + (size_t)dr * N + n) = __builtin_convertvector(v, bf16x4);
            }
        }
        __syncthreads();  // the sums are read: the rings may be filled for the next 16 tokens
    }
}

template <int EPI, int WR, int WAVES, class Gather>
hipError_t launch_shape(const bf16_t* a, Gather gather, const int32_t* offsets, const bf16_t* b0, const bf16_t* b1, bf16_t* c,
                        int slots, int S, int N, int K, hipStream_t st) {
    constexpr int BNO = EPI == kSwiglu ? WR / 2 : WR;
    constexpr int kLds = Shape<WR, WAVES>::LDS;
    // Where rows are not whole 128-byte lines every piece shares its lines with its neighbours, which other wavefronts load: no
    // non-temporal hint there (900 layers whose rows are none, weights from HBM, with the hint against without, by MiB of a
    // product's weights: 1 to 4 1.01, 8 to 64 1.02 to 1.03, 128 and more 1.03 to 1.05 of the time; one token, d 1992, f 13144, five
    // slots 175 / 201 us).
    const bool once = K % 64 == 0;
    auto kern = once ? few_gemm_bf16<EPI, WR, WAVES, true, Gather> : few_gemm_bf16<EPI, WR, WAVES, false, Gather>;
    static std::atomic<bool> attr_set[2] = {};  // set once per kernel; setting it twice from two threads is harmless
    if (!attr_set[once].load(std::memory_order_acquire)) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
        if (e != hipSuccess) return e;
        attr_set[once].store(true, std::memory_order_release);
    }
    const int n_units = (N + BNO - 1) / BNO;
    kern<<<(unsigned)(slots * n_units), 64 * WAVES, kLds, st>>>(a, gather, offsets, b0, b1, c, S, N, K, n_units);
    return hipGetLastError();
}

template <int EPI, class Gather>
hipError_t launch_one(const bf16_t* a, Gather gather, const int32_t* offsets, const bf16_t* b0, const bf16_t* b1, bf16_t* c,
                      int slots, int S, int N, int K, hipStream_t st) {
    DeviceShape shape;
    hipError_t e = device_shape(&shape);
    if (e != hipSuccess) return e;
    const long long units = (long long)slots * ((N + (EPI == kSwiglu ? 15 : 31)) / (EPI == kSwiglu ? 16 : 32));
    // Eight wavefronts only where each has a walk of some length (K 512, 128 workgroups: 4.6 / 5.4 us with four / eight).
    const bool long_k = K >= kLongK;
    if constexpr (EPI != kSwiglu) {
        if (2 * units <= shape.cus && long_k) return launch_shape<EPI, 16, 8>(a, gather, offsets, b0, b1, c, slots, S, N, K, st);
        if (2 * units <= shape.cus) return launch_shape<EPI, 16, 4>(a, gather, offsets, b0, b1, c, slots, S, N, K, st);
    }
    if (units <= shape.cus && long_k) return launch_shape<EPI, 32, 8>(a, gather, offsets, b0, b1, c, slots, S, N, K, st);
    // Short walks in many workgroups: what a workgroup waits for before its walk and after it counts, and 64 rows halve
    // their number (16 tokens, K 768, 1536 units of 32 rows 13.5 -> 11.5 us, K 1000, 6016 units 62.6 -> 56.6); with a long K 32
    // rows keep more weights in flight (K 4096, 1792 units of 16 + 16 rows: 71.5 against 73.7 us).  Up to K 512 that holds as
    // soon as 32 rows take more workgroups than the chip holds (513 to 1023 units, 64 against 32 rows: 0.87 of the time, and 0.96
    // with K 512 to 1024, slots without rows making it up to 1.17; 1.03 with K 1024 to 2048).
    if ((units > 2 * shape.cus && K <= kShortK) || (units >= 4 * shape.cus && K <= kLongK))
        return launch_shape<EPI, 64, 4>(a, gather, offsets, b0, b1, c, slots, S, N, K, st);
    return launch_shape<EPI, 32, 4>(a, gather, offsets, b0, b1, c, slots, S, N, K, st);
}

}  // namespace

// Whether a product of few tokens is faster in the streaming kernels: where weight rows are not whole 128-byte lines and the
// walk is long.  A load instruction takes time per line that it touches: 128 bytes of a row are two lines here, the
// streaming kernels' 256 bytes three, of token rows too, so it hangs on the rows per slot.  Measured at 1100 layers of K from 2048
// on, time here / streaming at 1 to 2, 3 to 4, 6, 8, 12 to 16 rows per slot: one matrix, 129 to 256 units 1.02, 1.08, 1.11, 1.11,
// 1.10; 257 to 512 0.96, 1.01, 1.00, 1.04, 1.06; 513 to 1024 0.95, 1.02, 1.05, 1.03, 1.07; above 0.90, 0.94, 0.94, 0.96, 1.04.
// SwiGLU, up to 256 units 0.72, 0.73, 0.73, 0.73, 0.74; 257 to 512 0.90, 0.94, 1.00, 1.02, 1.06; 513 to 768, where the streaming
// kernels' units of 32 + 32 rows make a round and a bit, 0.77, 0.82, 0.87, 0.88, 0.91; 769 to 1024 0.94, 1.04, 1.03, 1.04, 1.06; above
// 0.93, 0.95, 0.99, 1.01, 1.05.  (K 1024 to 2048: 0.94 to 0.97.)  Slots that stay empty, which the host does not know, cost the
// streaming kernels more.
bool few_product_streams(bool swiglu, long long A, int slots, int N, int K, int cus) {
    if (K % 64 == 0 || K < kLongK) return false;
    const long long units = (long long)slots * ((N + (swiglu ? 15 : 31)) / (swiglu ? 16 : 32));
    if (swiglu) return A > 6ll * slots && units > cus && (units <= 2 * cus || units > 3 * cus);
    if (units <= cus) return A > slots && 2 * units > cus;
    return A > (units <= 2 * cus ? 6ll : units <= 4 * cus ? 3ll : 8ll) * slots;
}

hipError_t launch_ffn_bf16_few(const emoe_layer_desc& d, const void* x_perm, SortingGather gather, const int32_t* offsets,
                               const void* w1, const void* w3, const void* w2, void* y_perm, void* ws, int passes,
                               hipStream_t st) {
    bf16_t* h = reinterpret_cast<bf16_t*>(static_cast<uint8_t*>(ws) + ffn_ws_layout(d).h);
    const bf16_t* xp = static_cast<const bf16_t*>(x_perm);
    const int A = d.T * d.k, slots = A < d.S ? A : d.S;
    DeviceShape shape;
    hipError_t e = device_shape(&shape);
    if (e != hipSuccess) return e;
    auto first = [&](auto rows) {
        const bf16_t* w1p = static_cast<const bf16_t*>(w1);
        if (d.act == EMOE_ACT_SWIGLU)
            return launch_one<kSwiglu>(xp, rows, offsets, w1p, static_cast<const bf16_t*>(w3), h, slots, d.S, d.d_ff, d.d_model, st);
        return launch_one<kRelu>(xp, rows, offsets, w1p, nullptr, h, slots, d.S, d.d_ff, d.d_model, st);
    };
    auto streamed = [&](int pass) { return launch_ffn_bf16_stream(d, x_perm, gather, offsets, w1, w3, w2, y_perm, ws, pass, st); };
    if (passes & 1) {
        if (few_product_streams(d.act == EMOE_ACT_SWIGLU, A, slots, d.d_ff, d.d_model, shape.cus)) e = streamed(1);
        else e = gather.sort.A > 0 ? first(gather) : first(RowGather(gather));
    }
    if (e != hipSuccess || !(passes & 2)) return e;
    if (few_product_streams(false, A, slots, d.d_model, d.d_ff, shape.cus)) return streamed(2);
    return launch_one<kPlain>(h, RowGather{nullptr, 1, 0, gather.out_perm}, offsets, static_cast<const bf16_t*>(w2), nullptr,
                              static_cast<bf16_t*>(y_perm), slots, d.S, d.d_model, d.d_ff, st);
}

}  // namespace emoe
