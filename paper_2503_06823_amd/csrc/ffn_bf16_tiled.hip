// Expert FFN for bf16 layers with many rows per slot: grouped GEMM on the gfx950 matrix cores
// (eMoE Section 1: the experts; Section 5.1: only resident, non-empty slots cost compute and
// memory reads).
//
//   pass 1: h[r, n]      = act(x_perm[r,:] . W1_s[n,:]) (* x_perm[r,:] . W3_s[n,:])   K = d_model
//   pass 2: y_perm[r, n] = h[r,:] . W2_s[n,:]                                         K = d_ff
//
// Tile: a workgroup of NW = 4 wavefronts (2 x 2, one per SIMD) owns 256 tokens x 256 weight rows;
// each wavefront accumulates 128 x 128 as 8 x 8 blocks of v_mfma_f32_16x16x32_bf16 in fp32 (256
// accumulator registers).  The kernel runs at the chip's power limit, and this shape does the most
// matrix work per joule: an instruction reads and writes its accumulators once per 32 K elements where
// the 32 x 32 x 16 shape does so per 16.  A loop of nothing but matrix instructions on N(0,1) operands
// runs at 2.08 PFLOP/s with it, at 1.83 with 32 x 32 x 16; with it the Mixtral prefill layer (4096
// tokens, 4 slots) takes 2.15 ms instead of 2.30, a fine-grained layer (d 2048, f 1408, 24 slots of
// 2048 rows) 0.79 instead of 0.83.  Eight wavefronts (128 x 64 each) measured slower: more LDS reads
// per MFMA.  In the SwiGLU pass the 256 weight rows are 128 rows of W1 and the SAME 128 rows of
// W3, arranged so that a lane holds the gate and the up value of the same output element and the
// activation is applied in registers.  The weight rows go on the MFMA's row operand: a lane then
// owns four consecutive output columns of one token in every block, which two exchanges between lanes
// turn into stores of eight (see epilogue()).
//
// Data movement: both operands are K-contiguous in memory.  K is walked in tiles of 64, so that a
// tile row is one whole 128-byte cache line (with 64-byte rows every line is requested twice, by
// consecutive K tiles; halving the requests to L2 was worth 8-15 % here, where the kernel runs at
// the chip's power limit).  An operand tile (256 rows x 128 bytes = 32 KiB) goes from global memory
// straight into LDS with buffer_load_dwordx4 ... lds (no staging registers, no LDS store
// instructions).  LDS is a ring of five operand tiles - weight rows of K tile t in slot 2t mod 5,
// token rows in slot 2t+1 mod 5 - so one and a half K tiles are in flight while one is multiplied.
// Each load instruction fills 1 KiB of LDS contiguously (8 rows x 128 bytes); the 16-byte chunk c
// of row r is stored at chunk position c ^ ((r >> 1) & 7), chosen by which global chunk a lane
// fetches, which makes the MFMA fragment reads (16 rows x four chunks per ds_read_b128) bank-conflict
// free without padding.  Buffer addressing gives a uniform (scalar) K offset plus a per-lane row
// offset, so the loop has no address arithmetic; in the K tail, chunks past K are fetched out of
// range and arrive as zeros.
//
// Schedule per K tile (two MFMA K-steps of 32 each): fragment reads for the next step, the loads
// of tile t+2 and the scalar arithmetic are slotted between the MFMAs, so no memory instruction waits in a full
// queue while the matrix pipe idles.  One barrier per tile, between its steps.  The places between two MFMAs are counted:
// an MFMA takes 16 cycles, every other instruction 4 or more, and with one wavefront per SIMD nobody else fills a gap.
// Fragment read, load and a piece of scalar arithmetic therefore each have a place of their own (the arithmetic in one lump of
// ten instructions and loads beside reads: fine-grained layer's products 430 + 260 us against 420 + 251; prefill 1297 + 634
// against 1276 + 626; 4096 tokens in four even slots).
//
// The stream of operand tiles does not stop between output tiles: an output tile's last two K tiles
// request the first two of the next one, and the epilogue stores from registers, without LDS and
// without a barrier (see epilogue()), so that they arrive meanwhile.  A wavefront's tile boundary used
// to cost 24 000 cycles (epilogue through LDS, then the first loads from nothing), a fifth of the
// fine-grained layer's first product (32 K tiles of 2 048 cycles per output tile); fine-grained layer
// 788 -> 763 us, Mixtral prefill layer 2153 -> 2095, two prompts at that shape 816 -> 802.
//
// Slots that do not fill their tiles: a slot's rows are spread evenly over its m-tiles in whole
// 16-row MFMA blocks (257 rows: tiles of 144 and 113 rows, not 256 and 1), a tile's blocks alternate
// between the two rows of wavefronts, and the K loop is compiled for 0 .. 8 blocks per wavefront, so
// that matrix work is done for blocks with rows only and both wavefront rows finish together.  A
// tile still costs a pass over its weight panel whatever it holds (8 slots of 257 rows at the Mixtral
// shape: 0.96 -> 0.88 ms; of 513 rows: 1.51 -> 1.41 ms; full tiles unchanged).
//
// Ragged groups: group sizes live on the device.  The launch is persistent (one workgroup per CU);
// every workgroup derives the list of (slot, m-tile, n-tile) tiles from slot_offsets and takes its
// share (see "work distribution" below).  Workgroup ids are dealt round-robin to the 8 XCDs, so
// ids are remapped: the workgroups of an XCD hold consecutive tiles of an order in which 32
// consecutive tiles form a block of 8 m-tiles x 4 n-tiles of one slot (see tile_in_slot), so that
// XCD's L2 supplies 12 operand panels for 32 tiles.
#include <atomic>
#include <type_traits>

#include "common.h"
#include "mfma_agpr.h"

namespace emoe {
namespace {

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void;
// a pointer into global memory, said so: the loads are counted by vmcnt alone (a flat load has to be waited for with vmcnt(0))
typedef const int32_t __attribute__((address_space(1)))* global_i32;

constexpr int BM = 256;                     // tokens per tile
constexpr int BR = 256;                     // weight rows per tile (SwiGLU: 128 of W1 + 128 of W3)
constexpr int BK = 64;                      // K elements per tile
constexpr int ROW_BYTES = BK * 2;           // 128: a tile row is one whole cache line
constexpr int TILE_BYTES = BM * ROW_BYTES;  // 32 KiB per operand
constexpr int SLOTS = 5;                    // LDS ring of operand tiles: w(t), x(t), w(t+1), x(t+1), w(t+2), ...
constexpr size_t LDS_BYTES = SLOTS * TILE_BYTES;  // 160 KiB, all of a CU's LDS
constexpr int KSTEP = 32;                   // K elements of one matrix instruction (16 x 16 x 32)
static_assert(BK / KSTEP == 2, "the K loop is written out for two MFMA K-steps per tile");
constexpr int kMaxSplits = 8;           // K pieces per leftover tile, at most
constexpr int kFixupGroups = (kMaxGroups - 1) * 16;  // workgroups of the fix-up launch: the most units there can be
constexpr int kPlanFloats = kTiledPlanBytes / 4;  // the plan sits ahead of the partial sums
constexpr unsigned kRotation = 21;  // K-tile rotation per slot
constexpr int kScalarPieces = 5;    // pieces of a step's address arithmetic
constexpr int NW = 4;            // wavefronts per workgroup, arranged 2 (tokens) x NW/2 (weight rows)
constexpr int WN = NW / 2;
constexpr int TS = 8;            // 16-token blocks per wavefront (128 tokens): the grain in which blocks without rows are skipped
constexpr int WB = BR / WN / 16; // 16-row weight blocks per wavefront
constexpr int RPI = 1024 / ROW_BYTES;      // tile rows filled by one load instruction (8)
constexpr int LPW = BM / RPI / NW;         // load instructions per wavefront, per tile and operand (8)

enum Epilogue { kPlain = 0, kSwiglu = 1, kRelu = 2 };

// s_waitcnt immediate: vmcnt <= n and all LDS traffic done (vmcnt[3:0] | [15:14], expcnt [6:4], lgkmcnt [11:8])
constexpr int wait_imm(int n) { return (n & 0xf) | ((n >> 4) << 14) | (0x7 << 4) | (0x0 << 8); }

// Workgroup barrier once at most `n` of this wavefront's global->LDS loads are still pending and
// all its LDS reads have returned.  __syncthreads() would drain every pending load (its release
// fence counts the LDS writes of the loads), which is exactly what the deep prefetch must avoid.
// The empty asm statements stop the compiler from moving LDS accesses across the barrier.
template <int N>
__device__ __forceinline__ void barrier_keep_loads() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(wait_imm(N));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}

// ---- work distribution ------------------------------------------------------------------------
// The launch is persistent: one workgroup per CU.  Output tiles are numbered in (slot, n-tile,
// m-tile) order of tile_in_slot.  The first `rounds * G` tiles are dealt out whole, `rounds` per
// workgroup, so that the 32 workgroups of an XCD hold 32 consecutive tiles at any time (one weight
// panel and the slot's token panels stay in that XCD's L2).  Round r covers tiles r*G .. (r+1)*G-1,
// 32 for each XCD: every XCD works its way through all slots, so slots whose tiles cost less (fewer
// rows than a tile holds) do not leave some XCDs idle while others still work (a contiguous range of
// tiles per XCD took 4-7 % longer at 250-500 rows per slot).  The `left` tiles that do not fill a
// round are split along K into `splits` pieces each, so that they too occupy (nearly) every CU: a
// piece writes its fp32 accumulators to the workspace and a small second kernel adds the pieces in
// order and applies the epilogue.  Everything is derived from slot_offsets on the device.
struct Plan {
    int tiles;   // output tiles in total
    int rounds;  // whole tiles per workgroup
    int left;    // tiles beyond rounds * G
    int splits;  // K pieces per leftover tile (1 = none)
};

__device__ __forceinline__ Plan make_plan(int tiles, int k_tiles, int G) {
    Plan p;
    p.tiles = tiles;
    p.rounds = p.tiles / G;
    p.left = p.tiles - p.rounds * G;
    int sp = p.left > 0 ? G / p.left : 1;
    const int by_k = k_tiles / 8;  // at least 8 K tiles (512 elements) per piece
    sp = sp < by_k ? sp : by_k;
    sp = sp > kMaxSplits ? kMaxSplits : sp;
    p.splits = sp < 1 ? 1 : sp;
    return p;
}

// Order of a slot's m_tiles x n_tiles output tiles.  The 32 workgroups of an XCD hold 32 consecutive
// tiles at any time and their L2 has to supply one operand panel per distinct m-tile and per
// distinct n-tile among them, so consecutive tiles should form compact blocks: the n-tiles are
// taken four at a time, and inside such a group of columns the m-tiles eight at a time, m fastest
// (12 panels for 32 tiles; m fastest over a whole tall slot would need up to 33).
// rem = number of the tile within the slot -> its m-tile and n-tile.
constexpr int kBlockM = 8, kBlockN = 4;
constexpr int kSkipBlocksUpToTiles = kBlockM;  // see the K loop's dispatch
__device__ __forceinline__ void tile_in_slot(int rem, int m_tiles, int n_tiles, int& mt, int& nt) {
    const int group = rem / (m_tiles * kBlockN);  // group of up to four n-tiles
    const int gn = n_tiles - group * kBlockN < kBlockN ? n_tiles - group * kBlockN : kBlockN;
    int r = rem - group * (m_tiles * kBlockN);
    const int full = m_tiles / kBlockM;           // whole blocks of eight m-tiles
    int mb = kBlockM, m0 = 0;
    if (r < full * kBlockM * gn) {
        m0 = (r / (kBlockM * gn)) * kBlockM;
        r %= kBlockM * gn;
    } else {
        r -= full * kBlockM * gn;
        m0 = full * kBlockM;
        mb = m_tiles - m0;
    }
    mt = m0 + r % mb;
    nt = group * kBlockN + r / mb;
}

// Rows per m-tile of a slot of `rows` rows cut into `tiles` tiles: the rows are spread evenly (in
// whole 16-row MFMA blocks), so that a slot of 257 rows becomes tiles of 144 and 113 rows instead of
// 256 and 1.  A tile costs a pass over its weight panel whatever it holds; what is saved is the
// matrix work of the blocks without rows, which both tiles then skip.
__device__ __forceinline__ int rows_per_tile(int rows, int tiles) {
    const int even = (rows + tiles - 1) / (tiles > 0 ? tiles : 1);
    return (even + 15) & ~15;  // <= BM, so tile number `tiles - 1` still starts inside the slot
}

// Which wavefronts multiply which of a tile's 16-row token blocks: the blocks alternate between
// the two wavefront rows, so that both finish together whatever the number of blocks that hold rows.
// -> first tile row of block j of wavefront row wm, and the number of its blocks that hold rows.
__device__ __forceinline__ int token_row(int wm, int j) { return (2 * j + wm) * 16; }
__device__ __forceinline__ int blocks_of_wavefront(int row0, int row_end, int wm) {
    return ((row_end - row0 + 15) / 16 - wm + 1) / 2;
}

// Four 16 x 16 output blocks of a wavefront side by side: 16-token block ts, weight blocks 4 wg .. 4 wg + 3.  `gate`
// holds the accumulators (for SwiGLU the gate rows), `up` the matching up rows (unused otherwise).
// A lane holds token lane%16 and weight rows 4*(lane/16) + 0..3 of each block.
template <int EPI>
__device__ __forceinline__ void epilogue_blocks(const floatx4 (&gate)[4], const floatx4 (&up)[4], bf16_t* __restrict__ c,
                                                const int32_t* __restrict__ out_perm, int row0, int row_end, int n0, int N,
                                                int wm, int wn, int ts, int wg, int lane) {
    constexpr int BNO = EPI == kSwiglu ? BR / 2 : BR;
    const int r = row0 + token_row(wm, ts) + (lane & 15);
    if (r >= row_end) return;
    bf16_t* crow = c + (size_t)((EPI == kPlain && out_perm != nullptr) ? out_perm[r] : r) * N;
    const int col0 = n0 + wn * (BNO / WN) + wg * 64 + (lane >> 4) * 4;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int n = col0 + 16 * b;
        if (n >= N) continue;
        floatx4 v;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float t = gate[b][q];
            if (EPI == kSwiglu) t = t / (1.0f + __expf(-t)) * up[b][q];
            if (EPI == kRelu) t = fmaxf(t, 0.0f);
            v[q] = t;
        }
        *reinterpret_cast<bf16x4*>(crow + n) = __builtin_convertvector(v, bf16x4);
    }
}

// The slot table in registers: lane s of every wavefront holds slot s's row range and the number of
// the first output tile of that slot, so that finding a tile's slot is one ballot and three lane
// reads instead of a walk over slot_offsets in memory (a few thousand cycles per tile).
struct SlotTable {
    int begin, end;  // rows of slot `lane`
    int tiles;       // m-tiles of slot `lane`
    int first;       // number of the slot's first output tile (exclusive prefix of tiles * n_tiles)
    int total;       // all output tiles (uniform)
};

__device__ __forceinline__ SlotTable make_slot_table(const int32_t* __restrict__ offsets, int S, int n_tiles, int lane) {
    SlotTable t;
    t.begin = lane < S ? offsets[lane] : 0;
    t.end = lane < S ? offsets[lane + 1] : 0;
    t.tiles = (t.end - t.begin + BM - 1) / BM;
    const int span = t.tiles * n_tiles;
    int incl = span;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int up = __shfl_up(incl, off);
        if (lane >= off) incl += up;
    }
    t.first = incl - span;
    t.total = __builtin_amdgcn_readlane(incl, 63);
    return t;
}

__device__ __forceinline__ void decode_tile(const SlotTable& t, int S, int n_tiles, int lane, int L, int& slot,
                                            int& row0, int& row_end, int& nt, int& slot_tiles) {
    // slots are in tile order and an empty slot starts where its successor does: the last slot that
    // starts at or before L is the non-empty one that holds it
    const unsigned long long m = __ballot(lane < S && t.first <= L);
    slot = __popcll(m) - 1;
    const int rem = L - __builtin_amdgcn_readlane(t.first, slot);
    const int tiles = __builtin_amdgcn_readlane(t.tiles, slot);
    int mt;
    tile_in_slot(rem, tiles, n_tiles, mt, nt);
    const int b = __builtin_amdgcn_readlane(t.begin, slot), e = __builtin_amdgcn_readlane(t.end, slot);
    const int rpt = rows_per_tile(e - b, tiles);
    row0 = b + mt * rpt;
    row_end = row0 + rpt < e ? row0 + rpt : e;
    slot_tiles = tiles;
}

// The value, through a statement that the compiler cannot look into.
__device__ __forceinline__ int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// Epilogue of a whole tile, straight from the registers: no LDS, no barrier, so that the next tile's operands can be on
// their way into the ring meanwhile.  The MFMA layout gives a lane four consecutive columns of one token in every block;
// two exchanges between odd and even rows of 16 lanes turn those of two neighbouring blocks into eight consecutive columns
// of one block, and a store instruction then writes 64 contiguous bytes of each of 16 token rows.
// TBLOCKS: the wavefront's 16-row token blocks that hold rows.
// Every wavefront issues kEpilogueStores<EPI> stores, whatever the tile holds (rows and columns that do not exist are
// addressed out of range, which writes nothing): the K loop counts on it, see there.  "Out of range" is the first byte
// past the output, c_bytes: all 16 bytes of such a store then lie past it (the host checks leave room for a row
// between the largest output and 2^32), and nothing depends on what becomes of an address that wraps.
template <int EPI>
constexpr int kEpilogueStores = TS * (EPI == kSwiglu ? WB / 2 : WB) / 2;

template <int EPI, int TBLOCKS>
__device__ __forceinline__ void epilogue(floatx4 (&acc)[WB][TS], __amdgpu_buffer_rsrc_t c_rsrc, uint32_t c_bytes, const int (&out_entry)[2],
                                         bool scatter, int row0, int row_end, int n0, int N, int wm, int wn, int lane) {
    constexpr int BNO = EPI == kSwiglu ? BR / 2 : BR;
    constexpr int NB = EPI == kSwiglu ? WB / 2 : WB;
    const int col0 = n0 + wn * (BNO / WN) + ((lane >> 4) & 1) * 16 + (lane >> 5) * 8;
#pragma unroll
    for (int ts = 0; ts < TS; ++ts) {
        const bool row_ok = row0 + token_row(wm, ts) + (lane & 15) < row_end;
        int r_out = row0 + token_row(wm, ts) + (lane & 15);
        if (scatter) r_out = __shfl(out_entry[ts >> 2], (ts & 3) * 16 + (lane & 15));  // the token's row of the output
        const uint32_t row_off = (uint32_t)r_out * (uint32_t)N * 2u;
#pragma unroll
        for (int np = 0; np < NB; np += 2) {
            uintx4 val = {0u, 0u, 0u, 0u};
            if (ts < TBLOCKS) {
                uint32_t two[2][2];  // block, its four columns as two packed pairs
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    const floatx4& gate = acc[np + b][ts];
                    const floatx4& up = acc[EPI == kSwiglu ? np + b + NB : np + b][ts];
                    floatx4 v;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        float t = acc_read(gate[q]);
                        if (EPI == kSwiglu) t = t * __builtin_amdgcn_rcpf(1.0f + __expf(-t)) * acc_read(up[q]);
                        if (EPI == kRelu) t = fmaxf(t, 0.0f);
                        v[q] = t;
                    }
                    const bf16x4 o = __builtin_convertvector(v, bf16x4);
                    __builtin_memcpy(two[b], &o, 8);
                }
                const auto lo = __builtin_amdgcn_permlane16_swap(two[0][0], two[1][0], false, false);
                const auto hi = __builtin_amdgcn_permlane16_swap(two[0][1], two[1][1], false, false);
                val = uintx4{lo[0], hi[0], lo[1], hi[1]};
            }
            const int n = col0 + np * 16;
            const uint32_t off = row_ok && n < N ? row_off + (uint32_t)n * 2u : c_bytes;
            __builtin_amdgcn_raw_buffer_store_b128(val, c_rsrc, (int)off, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);  // a few blocks at a time: the accumulators stay where they are until used
    }
}

template <int EPI, bool KTAIL>
__global__ __launch_bounds__(64 * NW) void grouped_gemm_bf16(const bf16_t* __restrict__ a, RowGather gather,
                                                         const int32_t* __restrict__ offsets,
                                                         const bf16_t* __restrict__ b0,
                                                         const bf16_t* __restrict__ b1, bf16_t* __restrict__ c,
                                                         float* __restrict__ partials, int c_rows, int S, int N, int K,
                                                         int n_tiles, int XCDS) {
    constexpr int BNO = EPI == kSwiglu ? BR / 2 : BR;  // output columns per tile
    extern __shared__ __align__(16) char lds[];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    // at least two: an item's last two K tiles request the first two of the next one (a second one past K is all zeros)
    const int k_tiles_all = K > BK ? (K + BK - 1) / BK : 2;
    const int G = gridDim.x;
    const SlotTable table = make_slot_table(offsets, S, n_tiles, lane);
    const Plan plan = make_plan(table.total, k_tiles_all, G);
    if (blockIdx.x == 0 && tid == 0)  // for the fix-up kernel, which then need not derive it again
        *reinterpret_cast<int4*>(partials) = make_int4(plan.tiles, plan.rounds, plan.left, plan.splits);
    const int rows_total = offsets[S];
    const int xcd = blockIdx.x % XCDS, cu = blockIdx.x / XCDS, per_xcd = G / XCDS;
    const int sk_item = xcd * per_xcd + cu;  // this workgroup's piece of the leftover tiles

    // ---- the tiles of this workgroup ---------------------------------------------------------------
    struct Item {
        int slot, row0, row_end, nt, slot_tiles;
        int kb, kt;  // its K tiles: kb .. kb + kt - 1
        int piece;   // -1: a whole tile; else the number of the K piece of a leftover tile (always the last item)
    };
    auto item_at = [&](int idx, Item& it) {
        int L;
        it.kb = 0;
        it.kt = k_tiles_all;
        it.piece = -1;
        if (idx < plan.rounds) {
            L = idx * G + xcd * per_xcd + cu;
        } else {
            if (idx > plan.rounds || sk_item >= plan.left * plan.splits) return false;
            L = plan.rounds * G + sk_item / plan.splits;
            if (plan.splits > 1) {
                const int sp = sk_item % plan.splits;
                it.kb = (int)((long long)k_tiles_all * sp / plan.splits);
                it.kt = (int)((long long)k_tiles_all * (sp + 1) / plan.splits) - it.kb;
                it.piece = sk_item;
            }
        }
        decode_tile(table, S, n_tiles, lane, L, it.slot, it.row0, it.row_end, it.nt, it.slot_tiles);
        return true;
    };

    // ---- global -> LDS -----------------------------------------------------------------------------
    // Wavefront w issues, per K tile and per operand, load instructions i = 0..LPW-1; instruction
    // (w, i) fills tile rows (LPW*w + i)*8 .. +7, 128 bytes each.  Lane l lands in row l>>3, chunk
    // position l&7 and therefore fetches global chunk (l&7) ^ ((row>>1)&7).
    const int l_row = lane >> 3;  // row within a load instruction's eight rows
    const int l_pos = lane & 7;   // chunk position within the row, in LDS
    const uint32_t a_bytes = (uint32_t)(gather.perm != nullptr ? gather.rows : rows_total) * (uint32_t)K * 2u;
    const uint32_t b_bytes = (uint32_t)N * (uint32_t)K * 2u;
    const __amdgpu_buffer_rsrc_t a_rsrc = make_rsrc(a, a_bytes);
    const uint32_t c_bytes = (uint32_t)c_rows * (uint32_t)N * 2u;
    const __amdgpu_buffer_rsrc_t c_rsrc = make_rsrc(c, c_bytes);
    const bf16_t* wsel = (EPI == kSwiglu && wave >= NW / 2) ? b1 : b0;  // upper wavefronts load the W3 half
    // that chunk depends on i only through its parity
    const int chunk2[2] = {l_pos ^ (l_row >> 1), l_pos ^ (4 + (l_row >> 1))};
    static_assert(RPI == 8 && LPW == 8, "the swizzle of a row is a function of l_row and the parity of i");
    // A wavefront loads 64 rows of a token tile: a lane looks up where row 64 wave + lane comes from (its perm entry,
    // or the row of x_perm itself), and the lanes that load pieces of it get the row from that lane.
    auto load_perm = [&](const Item& it) {
        int r = it.row0 + LPW * RPI * wave + lane;
        r = r >= it.row_end ? it.row_end - 1 : r;
        return gather.perm != nullptr ? global_i32(gather.perm)[r] : r;
    };
    const int perm_div = gather.perm != nullptr ? gather.k : 1;
    // (the lane number is made opaque where addresses are formed: the parts of them that are the same for every item would
    // otherwise be computed ahead of the loop, and there are no registers to keep them in)
    auto token_addr = [&](const Item& it, int perm_entry, uint32_t (&voff)[LPW]) {
        const int l = opaque(lane);
        const uint32_t x_row = (uint32_t)perm_entry / (uint32_t)perm_div;  // the token's row of x, not a copy of it
#pragma unroll
        for (int i = 0; i < LPW; ++i) {
            const int tr = (LPW * wave + i) * RPI + (l >> 3);
            const uint32_t row = (uint32_t)__shfl((int)x_row, i * RPI + (l >> 3));
            const int v = opaque((int)((row * (uint32_t)K + ((l & 7) ^ ((tr >> 1) & 7)) * 8) * 2u));  // (no branch around it)
            // rows past the slot's end: out of range, zeros without memory traffic
            voff[i] = it.row0 + tr >= it.row_end ? a_bytes : (uint32_t)v;
        }
    };
    auto weight_addr = [&](const Item& it, uint32_t (&voff)[LPW]) {
        const int l = opaque(lane);
#pragma unroll
        for (int i = 0; i < LPW; ++i) {
            const int tr = (LPW * wave + i) * RPI + (l >> 3);  // row of the tile
            int n = it.nt * BNO + (EPI == kSwiglu ? tr % (BR / 2) : tr);  // SwiGLU: second half = same rows of W3
            n = n < N ? n : N - 1;
            voff[i] = ((uint32_t)n * (uint32_t)K + ((l & 7) ^ ((tr >> 1) & 7)) * 8) * 2u;
        }
    };
    // Where an item's loads stand in its K tiles, as a byte offset into a row.  The tiles of different slots start at
    // different K tiles of their range and wrap around (all workgroups on the same 128-byte column of rows a power
    // of two apart land on few memory channels); the tiles of a slot share the start and so stay in step.  The order
    // is a fixed function of the tile.
    struct Cursor {
        int at, begin, end;
    };
    auto cursor_of = [&](const Item& it) {
        Cursor u;
        u.begin = it.kb * ROW_BYTES;
        u.end = u.begin + it.kt * ROW_BYTES;
        u.at = u.begin + __builtin_amdgcn_readfirstlane((int)(((unsigned)it.slot * kRotation) % (unsigned)it.kt)) * ROW_BYTES;
        return u;
    };
    auto advance = [](Cursor& u) {
        u.at += ROW_BYTES;
        u.at = u.at == u.end ? u.begin : u.at;
    };
    // one load instruction of the token tile or the weight tile at row byte k; rs: the LDS byte of the ring slot, and of this
    // wavefront's part of it
    const int wave_rs = LPW * 1024 * wave;
    const uint32_t k_bytes = (uint32_t)K * 2u;
    auto issue_x = [&](const uint32_t (&voff)[LPW], int i, int rs, int k) {
        uint32_t v = voff[i];
        if (KTAIL && (uint32_t)(k + chunk2[i & 1] * 16) >= k_bytes) v = a_bytes;  // past K: zeros
        __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rsrc, (lds_void*)(lds + rs + i * 1024), 16, (int)v, k, 0, 0);
    };
    auto issue_w = [&](const uint32_t (&voff)[LPW], const bf16_t* base, int i, int rs, int k, bool once) {
        uint32_t v = voff[i];
        if (KTAIL && (uint32_t)(k + chunk2[i & 1] * 16) >= k_bytes) v = b_bytes;
        lds_void* dst = (lds_void*)(lds + rs + i * 1024);
        if (once) __builtin_amdgcn_raw_ptr_buffer_load_lds(make_rsrc(base, b_bytes), dst, 16, (int)v, k, 0, 2);  // non-temporal hint
        else __builtin_amdgcn_raw_ptr_buffer_load_lds(make_rsrc(base, b_bytes), dst, 16, (int)v, k, 0, 0);
    };
    auto ring = [](int rs, int n) {  // the ring slot n places after the one at byte rs
        rs += n * TILE_BYTES;
        return rs >= SLOTS * TILE_BYTES ? rs - SLOTS * TILE_BYTES : rs;
    };

    // fragments: a lane holds row lane % 16 of a 16-row block and, in MFMA K-step kk, chunk 4 kk + lane / 16 of it.
    // The blocks of an operand are whole multiples of 16 rows apart, so they share the swizzle of the row; the places
    // of the two K-steps differ in bit 6 only.
    const int f_row = lane & 15;
    const int f_sw = ((lane >> 4) ^ ((f_row >> 1) & 7)) * 16;
    const int x_off = (token_row(wm, 0) + f_row) * ROW_BYTES + f_sw;  // token block 0 of this wavefront
    // SwiGLU: weight blocks 0..WB/2-1 are gate rows, WB/2..WB-1 the matching up rows
    const int w_off = (wn * ((EPI == kSwiglu ? BR / 2 : BR) / WN) + f_row) * ROW_BYTES + f_sw;

    // ---- prologue: K tiles 0 and 1 of the first item on their way, the first landed -------------------
    // Ring slots: the operand tiles follow each other round the ring, w(0), x(0), w(1), x(1), w(2), ...
    Item cur, nxt;
    if (!item_at(0, cur)) return;
    uint32_t a_voff[LPW], b_voff[LPW];
    int perm_entry = load_perm(cur);
    weight_addr(cur, b_voff);
    const bf16_t* w_base = wsel + (size_t)cur.slot * N * K;
    Cursor cursor = cursor_of(cur);
    int sw = 0;  // ring slot (LDS byte) of the weight rows of the K tile being multiplied
#pragma unroll
    for (int i = 0; i < LPW; ++i) issue_w(b_voff, w_base, i, wave_rs, cursor.at, false);
    token_addr(cur, perm_entry, a_voff);
#pragma unroll
    for (int i = 0; i < LPW; ++i) issue_x(a_voff, i, wave_rs + TILE_BYTES, cursor.at);
    advance(cursor);
#pragma unroll
    for (int i = 0; i < LPW; ++i) issue_w(b_voff, w_base, i, wave_rs + 2 * TILE_BYTES, cursor.at, false);
#pragma unroll
    for (int i = 0; i < LPW; ++i) issue_x(a_voff, i, wave_rs + 3 * TILE_BYTES, cursor.at);
    advance(cursor);
    barrier_keep_loads<2 * LPW>();
    bool stores_pending = false;  // the item before this one ended with kEpilogueStores<EPI> stores

    for (int idx = 0;; ++idx) {
        // the perm entries of the next item, which have this whole item to arrive in, and (with the combine folded in) the
        // output rows of this one: register h of a lane holds that of row 64 h + lane of this wavefront's 128
        const bool have_nxt = item_at(idx + 1, nxt);
        if (have_nxt) perm_entry = load_perm(nxt);
        int out_entry[2] = {0, 0};
        if (EPI == kPlain && gather.out_perm != nullptr) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int r = cur.row0 + token_row(wm, 4 * h + (lane >> 4)) + (lane & 15);
                out_entry[h] = global_i32(gather.out_perm)[r < cur.row_end ? r : cur.row_end - 1];
            }
        }

        // Everything that touches the matrix cores is compiled for NB = 0 .. TS token blocks: the number
        // of this wavefront's 16-row blocks that hold rows of the tile (a ragged or evenly cut tile holds
        // fewer than 256 rows).  NB = TS is the full tile, NB = 0 a wavefront that only takes part in the
        // loads and barriers.  The accumulators live and die inside one instance: where instances met, the compiler
        // would permute all 256 of them.
        auto do_item = [&](auto nb_c, auto once_c) {
            constexpr int NB = decltype(nb_c)::value;
            floatx4 acc[WB][TS];  // [weight block][token block]; an item's first MFMA step adds to nothing and need not clear them
            mfma_settle();  // the last of the item before have been read

            bf16x8 xf[2][TS], wf[2][WB];
            // fragment f of MFMA K-step kk: token blocks 0 .. NB - 1, then the weight blocks.  xp, wp: this lane's place (LDS
            // byte) in the operand tiles for that step
            auto load_frag = [&](int kk, int f, int xp, int wp) {
                if (f < NB) {
                    xf[kk][f] = *reinterpret_cast<const bf16x8*>(lds + xp + token_row(0, f) * ROW_BYTES);
                } else {
                    const int i = f - NB;
                    const int rr = (EPI == kSwiglu && i >= WB / 2) ? BR / 2 + (i - WB / 2) * 16 : i * 16;
                    wf[kk][i] = *reinterpret_cast<const bf16x8*>(lds + wp + rr * ROW_BYTES);
                }
            };
            // One MFMA K-step: multiplies the fragments of step kk and, slotted in between so that no memory
            // instruction waits in a full queue while the matrix pipe idles, reads the fragments of the step after it
            // (from xp, wp; in the first three quarters of the step, so that they are there at its end), issues LPW
            // global->LDS loads and runs `scalar`, the next step's address arithmetic, in kScalarPieces pieces.
            // A full tile reads a fragment after every third MFMA, and the others have places between those.  A tile with
            // fewer blocks is bound by when its operands arrive, not by the matrix pipe: up to six blocks, step 1's
            // loads go out in its first half (8 slots of 160 rows at the Mixtral shape: 371 + 186 -> 345 + 171 us with the
            // order of the operands in the ring; on full tiles 1 % slower).
            auto step = [&](auto first_c, int kk, int xp, int wp, auto issue, auto scalar) {
                constexpr int MF = WB * NB, FR = WB + NB;
                if constexpr (NB == 0) {
    #pragma unroll
                    for (int i = 0; i < LPW; ++i) issue(i);
    #pragma unroll
                    for (int p = 0; p < kScalarPieces; ++p) scalar(p);
                } else {
                    constexpr auto frags_by = [](int m) { return m * FR / (MF * 3 / 4) < FR ? m * FR / (MF * 3 / 4) : FR; };
                    constexpr auto load_after = [](int i, int kk) {  // the MFMA behind which load i goes out
                        const int every = NB <= 6 && NB > 1 && kk == 1 ? MF / LPW / 2 : MF / LPW;
                        return NB == TS ? 7 + 6 * i : every * i + every / 2;
                    };
                    constexpr auto piece_after = [](int p) { return NB == TS ? 16 + 6 * p : MF / 8 + p * (MF * 3 / 4) / kScalarPieces; };
                    static_assert(frags_by(MF) == FR && load_after(LPW - 1, 0) < MF && piece_after(kScalarPieces - 1) < MF, "everything finds its place");
    #pragma unroll
                    for (int m = 0; m < MF; ++m) {
                        const int ni = m / NB;
                        const int mi = (ni & 1) ? NB - 1 - m % NB : m % NB;  // back and forth: only one operand changes between two MFMAs
                        if (decltype(first_c)::value) mfma_16x16x32_first(acc[ni][mi], wf[kk][ni], xf[kk][mi]);
                        else mfma_16x16x32(acc[ni][mi], wf[kk][ni], xf[kk][mi]);
    #pragma unroll
                        for (int f = frags_by(m); f < frags_by(m + 1); ++f) load_frag(kk ^ 1, f, xp, wp);
    #pragma unroll
                        for (int i = 0; i < LPW; ++i)
                            if (m == load_after(i, kk)) issue(i);
    #pragma unroll
                        for (int p = 0; p < kScalarPieces; ++p)
                            if (m == piece_after(p)) {
                                __builtin_amdgcn_sched_barrier(0);
                                scalar(p);
                                __builtin_amdgcn_sched_barrier(0);
                            }
                    }
                }
            };

            // ---- main loop -----------------------------------------------------------------------------
            // Per K tile: two MFMA steps of 32.  Weight rows of tile t+2 are requested during step 0 (into the slot
            // that held the token rows of tile t-1), token rows of tile t+2 during step 1 (into the slot of this
            // tile's weight rows, dead after the barrier): the weights, which come from HBM, have half a K tile longer to
            // arrive in than the token rows, which mostly come from nearer.  One barrier per tile, between the steps: by then every
            // wavefront has read its last fragments of tile t, and tile t+1 has landed once only the LPW newest
            // loads (weight rows of t+2) are pending - and, in an item's first K tile, the stores of the item before,
            // which are newer than the loads of this item's first two K tiles.
            // The stream of operand tiles does not end with the item: its last two K tiles request the first two of
            // the next one, which have the epilogue's time to arrive in.
            // A wavefront skips the fragment reads and MFMAs of its token blocks without rows: the kernel
            // runs at the chip's power limit, so work not done is speed for the others.
            int xp0 = ring(sw, 1) + x_off, wp0 = sw + w_off;
    #pragma unroll
            for (int f = 0; NB > 0 && f < NB + WB; ++f) load_frag(0, f, xp0, wp0);
            int xp1 = xp0 ^ 64, wp1 = wp0 ^ 64;
            int rs0 = ring(sw, 4) + wave_rs;
            __builtin_amdgcn_sched_barrier(0);
            auto k_tile = [&](auto first_c) {
                const int k = __builtin_amdgcn_readfirstlane(cursor.at);  // (uniform, which the compiler does not see)
                int sw1 = 0, sx1 = 0, rs1 = 0;
                step(first_c, 0, xp1, wp1, [&](int i) { issue_w(b_voff, w_base, i, rs0, k, decltype(once_c)::value); },
                     [&](int p) {
                         if (p == 0) sw1 = ring(sw, 2);
                         if (p == 1) wp0 = sw1 + w_off;
                         if (p == 2) sx1 = ring(sw, 3);
                         if (p == 3) xp0 = sx1 + x_off;
                         if (p == 4) rs1 = sw + wave_rs;
                     });
                __builtin_amdgcn_sched_barrier(0);
                if (stores_pending) {
                    barrier_keep_loads<LPW + kEpilogueStores<EPI>>();
                    stores_pending = false;
                } else {
                    barrier_keep_loads<LPW>();
                }
                __builtin_amdgcn_sched_barrier(0);
                step(std::false_type{}, 1, xp0, wp0, [&](int i) { issue_x(a_voff, i, rs1, k); },
                     [&](int p) {
                         if (p == 0) xp1 = xp0 ^ 64;
                         if (p == 1) wp1 = wp0 ^ 64;
                         if (p == 2) rs0 = ring(sw, 1);
                         if (p == 3) rs0 += wave_rs;
                         if (p == 4) advance(cursor);
                     });
                __builtin_amdgcn_sched_barrier(0);
                sw = sw1;
            };
            // the last two K tiles request the next item's first two
            auto turn_to_next = [&] {
                cursor = Cursor{0, 0, 2 * ROW_BYTES};
                if (have_nxt) {
                    token_addr(nxt, perm_entry, a_voff);
                    weight_addr(nxt, b_voff);
                    w_base = wsel + (size_t)nxt.slot * N * K;
                    cursor = cursor_of(nxt);
                } else {  // none: they go on, out of range: zeros land in ring slots that nobody reads any more
    #pragma unroll
                    for (int i = 0; i < LPW; ++i) { a_voff[i] = a_bytes; b_voff[i] = b_bytes; }
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            if (cur.kt == 2) {
                __builtin_amdgcn_s_waitcnt(wait_imm(0));  // nothing has waited for the next item's perm entries yet
                turn_to_next();
            }
            k_tile(std::true_type{});
    #pragma unroll 1
            for (int left = cur.kt - 1; left > 0; --left) {
                if (left == 2) turn_to_next();
                k_tile(std::false_type{});
            }
            mfma_settle();

            if (cur.piece < 0) {
                epilogue<EPI, NB>(acc, c_rsrc, c_bytes, out_entry, EPI == kPlain && gather.out_perm != nullptr, cur.row0, cur.row_end, cur.nt * BNO, N, wm, wn, lane);
            } else {  // a K piece of a leftover tile: raw accumulators to the workspace, [register][thread]
                float* dst = partials + kPlanFloats + (size_t)cur.piece * (BM * BR) + tid;
    #pragma unroll
                for (int i = 0; i < WB; ++i)
    #pragma unroll
                    for (int j = 0; j < NB; ++j) {  // (the fix-up skips blocks without rows)
    #pragma unroll
                        for (int v = 0; v < 4; ++v) dst[((i * TS + j) * 4 + v) * (64 * NW)] = acc_read(acc[i][j][v]);
                    }
            }
        };
        // Blocks without rows are skipped in slots of up to kBlockM tiles (one block of tile_in_slot), where a
        // tile's padding is a large share of the slot's matrix work.  In a taller slot the one ragged tile
        // multiplies its padding: the workgroups of an XCD share operand panels through L2 only while they
        // walk K in step, and a tile that finishes early falls out of step for good.  Skipping everywhere
        // fetches 5.4 instead of 3.15 GB from beyond L2 in the prefill layer's first product (Mixtral-8x22B
        // shape: 10.5 instead of 6.6 GB) and gains nothing: with the three policies (limit 4, 8, none) run
        // in turns inside one process, layer times differ by less than 1 % on every workload (prefill
        // 2.298 / 2.288 / 2.307 ms, fine-grained layer 0.845 / 0.842 / 0.836 ms).
        const int my_blocks = cur.slot_tiles > kSkipBlocksUpToTiles ? TS : blocks_of_wavefront(cur.row0, cur.row_end, wm);
        static_assert(TS == 8, "written out for eight token blocks per wavefront");
        // A slot of one m-tile: nobody else reads its weight panel, which is then loaded with the
        // non-temporal hint, so that the stream does not push the token rows out of the caches (but not with a K tail: rows are
        // not whole lines then, and a line between two K tiles would come from HBM twice).
        if (!KTAIL && cur.slot_tiles == 1) {
            if (my_blocks >= 8) do_item(std::integral_constant<int, 8>{}, std::true_type{});
            else if (my_blocks == 7) do_item(std::integral_constant<int, 7>{}, std::true_type{});
            else if (my_blocks == 6) do_item(std::integral_constant<int, 6>{}, std::true_type{});
            else if (my_blocks == 5) do_item(std::integral_constant<int, 5>{}, std::true_type{});
            else if (my_blocks == 4) do_item(std::integral_constant<int, 4>{}, std::true_type{});
            else if (my_blocks == 3) do_item(std::integral_constant<int, 3>{}, std::true_type{});
            else if (my_blocks == 2) do_item(std::integral_constant<int, 2>{}, std::true_type{});
            else if (my_blocks == 1) do_item(std::integral_constant<int, 1>{}, std::true_type{});
            else do_item(std::integral_constant<int, 0>{}, std::true_type{});
        } else {
            if (my_blocks >= 8) do_item(std::integral_constant<int, 8>{}, std::false_type{});
            else if (my_blocks == 7) do_item(std::integral_constant<int, 7>{}, std::false_type{});
            else if (my_blocks == 6) do_item(std::integral_constant<int, 6>{}, std::false_type{});
            else if (my_blocks == 5) do_item(std::integral_constant<int, 5>{}, std::false_type{});
            else if (my_blocks == 4) do_item(std::integral_constant<int, 4>{}, std::false_type{});
            else if (my_blocks == 3) do_item(std::integral_constant<int, 3>{}, std::false_type{});
            else if (my_blocks == 2) do_item(std::integral_constant<int, 2>{}, std::false_type{});
            else if (my_blocks == 1) do_item(std::integral_constant<int, 1>{}, std::false_type{});
            else do_item(std::integral_constant<int, 0>{}, std::false_type{});
        }
        if (!have_nxt) break;
        stores_pending = true;  // (a K piece is always the last item)
        cur = nxt;
    }
    // the surplus loads must not outlive the workgroup's LDS
    barrier_keep_loads<0>();
}

// Adds the K pieces of each leftover tile in piece order and applies the epilogue.  One unit of work
// per (leftover tile, 16 x 64 block position of the wavefronts), so the sum itself is spread over
// the chip.  The plan (how many leftover tiles, how many pieces)
// is read from the head of the workspace, where the main kernel left it: when nothing was split,
// which the host cannot know, every workgroup exits after one load.
constexpr int kFixupUnitsPerGroup = 4;  // units per workgroup of the fix-up launch, one per 64 * NW threads
template <int EPI>
__global__ __launch_bounds__(64 * NW * kFixupUnitsPerGroup) void splitk_fixup(const int32_t* __restrict__ offsets, bf16_t* __restrict__ c,
                                                        const int32_t* __restrict__ out_perm,
                                                        const int* __restrict__ hdr,
                                                        const float* __restrict__ partials, int S, int N, int K,
                                                        int n_tiles, int G) {
    constexpr int BNO = EPI == kSwiglu ? BR / 2 : BR;
    constexpr int NG = (EPI == kSwiglu ? WB / 2 : WB) / 4;  // groups of four output blocks
    constexpr int UNITS = TS * NG;
    Plan plan;  // uniform address: scalar loads
    plan.tiles = hdr[0]; plan.rounds = hdr[1]; plan.left = hdr[2]; plan.splits = hdr[3];
    if (plan.splits <= 1) return;
    // a workgroup holds kFixupUnitsPerGroup independent units (there is no barrier in this kernel): when nothing was
    // cut, which is the common case, a quarter as many workgroups have to start only to find that out
    const int tid = threadIdx.x % (64 * NW), lane = tid & 63, wave = tid >> 6;
    const int u = blockIdx.x * kFixupUnitsPerGroup + threadIdx.x / (64 * NW);  // the launch covers the most units there can be
    if (u >= plan.left * UNITS) return;
    const int tile = u / UNITS, unit = u % UNITS;
    const int ts = unit / NG, wg = unit % NG;
    int slot, row0, row_end, nt, slot_tiles;
    // the slot table in registers, as in the main kernel: a walk over slot_offsets in memory is a chain of up to S
    // dependent loads, longer than everything else this kernel does
    const SlotTable table = make_slot_table(offsets, S, n_tiles, lane);
    decode_tile(table, S, n_tiles, lane, plan.rounds * G + tile, slot, row0, row_end, nt, slot_tiles);
    if (row0 + token_row(wave / WN, ts) >= row_end) return;  // this wavefront's block holds no rows: nothing was written
    floatx4 gate[4], up[4];
#pragma unroll
    for (int v = 0; v < 16; ++v) { gate[v >> 2][v & 3] = 0.0f; up[v >> 2][v & 3] = 0.0f; }
    for (int sp = 0; sp < plan.splits; ++sp) {
        const float* src = partials + (size_t)(tile * plan.splits + sp) * (BM * BR) + tid;
        float g[16], w[16];  // all loads of a piece in flight together, then the adds
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int ni = wg * 4 + (v >> 2);
            g[v] = src[((ni * TS + ts) * 4 + (v & 3)) * (64 * NW)];
            w[v] = EPI == kSwiglu ? src[(((ni + WB / 2) * TS + ts) * 4 + (v & 3)) * (64 * NW)] : 0.0f;
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            gate[v >> 2][v & 3] += g[v];
            up[v >> 2][v & 3] += w[v];
        }
    }
    epilogue_blocks<EPI>(gate, up, c, out_perm, row0, row_end, nt * BNO, N, wave / WN, wave % WN, ts, wg, lane);
}

template <int EPI, bool KTAIL>
hipError_t launch_cfg(const bf16_t* a, RowGather gather, const int32_t* offsets, const bf16_t* b0, const bf16_t* b1, bf16_t* c,
                      float* partials, int c_rows, int S, int N, int K, int n_tiles, hipStream_t st) {
    auto kern = grouped_gemm_bf16<EPI, KTAIL>;
    static std::atomic<bool> attr_set{false};  // set once per kernel; setting it twice from two threads is harmless
    if (!attr_set.load(std::memory_order_acquire)) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS_BYTES);
        if (e != hipSuccess) return e;
        attr_set.store(true, std::memory_order_release);
    }
    DeviceShape shape;
    hipError_t es = device_shape(&shape);
    if (es != hipSuccess) return es;
    // persistent: one workgroup per CU (the partial sums of the tiles cut along K are sized for kMaxGroups)
    kern<<<shape.groups, 64 * NW, LDS_BYTES, st>>>(a, gather, offsets, b0, b1, c, partials, c_rows, S, N, K, n_tiles, shape.xcds);
    splitk_fixup<EPI><<<kFixupGroups / kFixupUnitsPerGroup, 64 * NW * kFixupUnitsPerGroup, 0, st>>>(offsets, c, gather.out_perm, reinterpret_cast<const int*>(partials),
                                                        partials + kPlanFloats, S, N, K, n_tiles, shape.groups);
    return hipGetLastError();
}

template <int EPI>
hipError_t launch_one(const bf16_t* a, RowGather gather, const int32_t* offsets, const bf16_t* b0, const bf16_t* b1, bf16_t* c,
                      float* partials, int c_rows, int S, int N, int K, hipStream_t st) {
    constexpr int BNO = EPI == kSwiglu ? BR / 2 : BR;
    const int n_tiles = (N + BNO - 1) / BNO;
    if (K % BK == 0 && K > BK) return launch_cfg<EPI, false>(a, gather, offsets, b0, b1, c, partials, c_rows, S, N, K, n_tiles, st);
    return launch_cfg<EPI, true>(a, gather, offsets, b0, b1, c, partials, c_rows, S, N, K, n_tiles, st);
}

}  // namespace

hipError_t launch_ffn_bf16_tiled(const emoe_layer_desc& d, const void* x_perm, RowGather gather,
                                 const int32_t* offsets,
                                 const void* w1, const void* w3, const void* w2, void* y_perm, void* ws,
                                 int passes, hipStream_t st) {
    const FfnWs lay = ffn_ws_layout(d);
    bf16_t* h = reinterpret_cast<bf16_t*>(static_cast<uint8_t*>(ws) + lay.h);
    float* partials = reinterpret_cast<float*>(static_cast<uint8_t*>(ws) + lay.partials);
    const bf16_t* xp = static_cast<const bf16_t*>(x_perm);
    const int A = d.T * d.k;  // rows of h and of y_perm; with the combine folded in (k = 1) of the layer's output
    hipError_t e = hipSuccess;
    if (!(passes & 1)) {
    } else if (d.act == EMOE_ACT_SWIGLU)
        e = launch_one<kSwiglu>(xp, gather, offsets, static_cast<const bf16_t*>(w1), static_cast<const bf16_t*>(w3), h,
                                partials, A, d.S, d.d_ff, d.d_model, st);
    else
        e = launch_one<kRelu>(xp, gather, offsets, static_cast<const bf16_t*>(w1), nullptr, h, partials, A, d.S, d.d_ff, d.d_model,
                              st);
    if (e != hipSuccess || !(passes & 2)) return e;
    return launch_one<kPlain>(h, RowGather{nullptr, 1, 0, gather.out_perm}, offsets, static_cast<const bf16_t*>(w2), nullptr, static_cast<bf16_t*>(y_perm),
                              partials, A, d.S, d.d_model, d.d_ff, st);
}

}  // namespace emoe
