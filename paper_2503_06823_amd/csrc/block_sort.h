// The stable counting sort of at most kBlockSortMax assignments by slot, done by every workgroup of a first product for
// itself (eMoE Section 3.2.2: the rows per slot are the experts' workload).
//
// A sort launch of its own costs a layer of few tokens some 4 us, as much as its gate, while a workgroup of the first product
// waits for two dependent reads anyway: the slots' offsets, then its rows' perm entries.  Here it reads the assignments
// instead, a dependent read less, and ranks them in some 600 cycles.  64 tokens, d 128, f 256, fp32: layer 21.3 -> 18.8 us; one token, d 4096, f 14336
// 116.8 -> 115.8; random layers of 1 to 90 tokens 1.00 to 1.24 times as fast.
//
// The wavefronts rank 64 assignments per pass with six ballots (one per bit of the slot id) and leave their counts in LDS;
// then every wavefront adds them up for itself, lane = slot.
#pragma once
#include "common.h"

namespace emoe {
namespace {

// The assignments of this wavefront with the same key as this lane's: the lanes that hold them.  One ballot per bit of the
// key, not one per slot.
static_assert(kMaxExperts == 64, "six bits of key");
__device__ __forceinline__ unsigned long long same_key(int key) {
    unsigned long long m = __ballot(key >= 0);
#pragma unroll
    for (int b = 0; b < 6; ++b) {
        const bool bit = (key >> b) & 1;
        const unsigned long long set = __ballot(bit);
        m &= bit ? set : ~set;
    }
    return m;
}

constexpr int kSortShares = kBlockSortMax / 64;                                        // of 64 assignments
constexpr int kSortLdsBytes = kSortShares * kMaxExperts * (int)sizeof(int);            // 4 KiB

template <int WAVES>
struct BlockSort {
    static constexpr int PASSES = kSortShares / WAVES;
    int begin, end;     // lane s: rows of slot s
    // slot << 16 | row of assignment assignment(p), -1: none.  One register an assignment: they live until the rows are listed,
    // and slot and row apart spilled the fp32 SwiGLU product, which holds 128 registers.
    int place[PASSES];

    __device__ static int assignment(int p) { return p * WAVES * 64 + (int)threadIdx.x; }

    // counts: kSortLdsBytes of LDS, free again after the caller's next barrier
    __device__ __forceinline__ void run(const SortTables& t, int S, int* counts) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        const unsigned long long below = (1ull << lane) - 1ull;
        const int slot_of_lane = lane < t.E ? t.slot_of_expert[lane] : -1;
        int e[PASSES], key[PASSES], rank[PASSES];
#pragma unroll
        for (int p = 0; p < PASSES; ++p) e[p] = assignment(p) < t.A ? t.topk_expert[assignment(p)] : -1;
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int s = __shfl(slot_of_lane, e[p] & 63);
            key[p] = (e[p] >= 0 && e[p] < t.E && s >= 0 && s < S) ? s : -1;
            rank[p] = 0;
            counts[(p * WAVES + wave) * kMaxExperts + lane] = 0;  // this wavefront's own row
        }
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            if (p * WAVES * 64 >= t.A) break;  // (uniform)
            const unsigned long long m = same_key(key[p]);
            rank[p] = __popcll(m & below);
            if (key[p] >= 0 && rank[p] == 0) counts[(p * WAVES + wave) * kMaxExperts + key[p]] = __popcll(m);
        }
        __syncthreads();
        // lane = slot: its total, and what comes before this wavefront's share of each pass
        int total = 0, before[PASSES];
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            before[p] = 0;
            if (p * WAVES * 64 >= t.A) continue;  // (uniform)
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                if (w == wave) before[p] = total;
                total += counts[(p * WAVES + w) * kMaxExperts + lane];
            }
        }
        int incl = total;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int up = __shfl_up(incl, off);
            if (lane >= off) incl += up;
        }
        begin = incl - total;
        end = incl;
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int row = __shfl(begin + before[p], key[p] & 63) + rank[p];
            place[p] = key[p] >= 0 ? key[p] << 16 | row : -1;
        }
    }

    // By one workgroup of the launch: the slots' sizes and offsets, and the assignments without a resident expert (only
    // possible when the caller broke emoe_route's precondition), which appear in no slot.
    __device__ __forceinline__ void store_slots(const SortTables& t, int S) const {
        const int lane = threadIdx.x & 63;
        if (threadIdx.x < 64) {
            if (lane < S) {
                t.slot_counts[lane] = end - begin;
                t.slot_offsets[lane] = begin;
            }
            if (lane == S - 1) t.slot_offsets[S] = end;
        }
#pragma unroll
        for (int p = 0; p < PASSES; ++p)
            if (place[p] < 0 && assignment(p) < t.A) t.inv_perm[assignment(p)] = -1;
    }

    // By one workgroup per tile of rows: the entries of rows row0 .. row0 + n - 1 of `slot`.
    __device__ __forceinline__ void store_rows(const SortTables& t, int slot, int row0, int n) const {
#pragma unroll
        for (int p = 0; p < PASSES; ++p)
            if (at(p, slot, row0) < (unsigned)n) {
                const int row = place[p] & 0xffff;
                t.perm[row] = assignment(p);
                t.inv_perm[assignment(p)] = row;
            }
    }

    // The same rows' assignments into `list` (LDS), between two barriers of the caller.
    __device__ __forceinline__ void list_rows(int slot, int row0, int n, int* list) const {
#pragma unroll
        for (int p = 0; p < PASSES; ++p)
            if (at(p, slot, row0) < (unsigned)n) list[at(p, slot, row0)] = assignment(p);
    }

    // Where assignment(p) is among the rows of `slot` from row0 on; past all of them if it is none of these.
    __device__ __forceinline__ unsigned at(int p, int slot, int row0) const { return (unsigned)(place[p] - (slot << 16 | row0)); }
};

}  // namespace
}  // namespace emoe
