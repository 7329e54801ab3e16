// How the kernel of the 64- and 128-row token tiles divides a product among the workgroups: arithmetic on sizes and nothing
// else, in constant expressions, so that the device and the host (the tests) evaluate the same text.
#pragma once

namespace emoe {
namespace mid {

constexpr int kMinShare = 8;    // K tiles per workgroup, at least, when tiles are cut
constexpr int kMinSpared = 48;  // tiles are cut only if that shortens every workgroup's K walk by this many K tiles

// Tiles cut along K: all tiles' K tiles, in tile order, are one sequence of `units`, and `sharers` workgroups take equal
// consecutive shares of it.  sharers == 0: nothing is cut.
struct Cut {
    unsigned units;
    int sharers;
};
// `tiles` output tiles of `kt` K tiles each, G workgroups.  Cutting pays when it spares every workgroup a K walk of some length: the
// pieces are extra traffic and the second kernel has work to do (a fine-grained layer with K = 2048, 176 tiles: 57 -> 72 us
// when cut regardless).  In 32 bits: fewer tiles than workgroups, 255 at most, of 2^22 K tiles at most (a slot's weight matrix
// has less than 2^31 elements in 8 columns or more).
constexpr Cut make_cut(int tiles, int kt, int G) {
    if (tiles >= G || tiles == 0) return Cut{0, 0};
    const unsigned units = (unsigned)tiles * (unsigned)kt;
    unsigned p = units / kMinShare;
    p = p < (unsigned)G ? p : (unsigned)G;
    const int share = p > 0 ? (int)((units + p - 1) / p) : 0;
    return Cut{units, ((int)p > tiles && kt - share >= kMinSpared) ? (int)p : 0};
}
// First unit of share g: units * g / sharers, rounded down, by parts that fit 32 bits.  Share g (0 .. sharers - 1) is
// [share_begin(g), share_begin(g + 1)); from `sharers` on shares are empty.
constexpr unsigned share_begin(Cut cut, int g) {
    if (g >= cut.sharers) return cut.units;
    const unsigned p = (unsigned)cut.sharers, whole = cut.units / p, rest = cut.units - whole * p;
    return whole * (unsigned)g + rest * (unsigned)g / p;
}
// The shares that hold a part of a tile: first .. end - 1, in K order.  More than one: the tile is cut.
struct Pieces {
    int first, end;
};
constexpr Pieces pieces_of(Cut cut, int tiles, int kt, int tile) {
    const unsigned begin = (unsigned)tile * (unsigned)kt;
    int first = tile * cut.sharers / tiles, end = (tile + 1) * cut.sharers / tiles;  // begin at or before the tile, and at or before its end
    if (share_begin(cut, first + 1) <= begin) ++first;
    if (share_begin(cut, end) < begin + (unsigned)kt) ++end;
    return Pieces{first, end};
}

// The first tile that begins in share g or after it.  No share holds the beginnings of two.
constexpr int first_tile(Cut cut, int kt, int g) { return (int)((share_begin(cut, g) + (unsigned)kt - 1) / (unsigned)kt); }

// ---- which tiles a product takes ---------------------------------------------------------------------
constexpr int kTileK = 64;                // K elements per K tile
constexpr long long kRowsPerSlot64 = 48;  // up to that many rows per slot on average: token tiles of 64 rows
constexpr int kMinPersistK = 64;          // K tiles from which on the persistent launch (which may cut) is used at all
constexpr int kNarrowFromK = 17;          // K tiles from which on column tiles may be narrower than a tile can hold

// Token rows and weight rows of a tile (SwiGLU: half of them rows of W1, half the same rows of W3), and whether the launch is a persistent one.
struct Arrangement {
    int rows, weight_rows;
    bool persist;
};
constexpr int k_tiles_of(int K) { return (K + kTileK - 1) / kTileK; }
// every slot adds at most one partial m-tile to the A / rows whole ones
constexpr long long most_m_tiles(long long A, int S, int rows) { return A / rows + (S < A ? S : A); }
// A assignments in S slots, N columns, K inputs.
// Tiles of 256 weight rows, unless they would leave CUs without a tile (the second product of a
// layer with a small d_model): then 128 weight rows and five stages, so that twice as many CUs
// stream weights, each with as many bytes in flight; and if K is long, in a persistent launch
// that cuts the tiles along K when even they are clearly fewer than the CUs (with a short K that
// never pays, and the second kernel's launch is saved).
// Few rows per slot: token tiles of 64 rows leave LDS for more stages, 96 (80 with 128 weight rows) KiB
// of weights in flight per CU instead of 64.  (With SwiGLU and 128 weight rows a wavefront of the
// 64-row arrangement would hold half a block of gate rows: that combination keeps 128 token rows.)
constexpr Arrangement arrangement(bool swiglu, long long A, int S, int N, int K, int cus) {
    const int widest = swiglu ? 128 : 256;
    const long long m_tiles = most_m_tiles(A, S, 128);
    const bool few_rows = A <= kRowsPerSlot64 * S;
    if (m_tiles * ((N + widest - 1) / widest) > cus) return Arrangement{few_rows ? 64 : 128, 256, false};
    const bool persist = k_tiles_of(K) >= kMinPersistK;
    // a short K (no cutting) and so few 128-row tiles that they leave a quarter of the CUs idle even
    // if every slot has a partial tile: 64-row tiles, about twice as many
    const bool underfilled = !persist && m_tiles * ((N + 127) / 128) <= cus * 3 / 4;
    return Arrangement{!swiglu && (few_rows || underfilled) ? 64 : 128, 128, persist};
}

// The workgroups of a launch that is not a persistent one, for at most m_tiles m-tiles of n column tiles each.  The kernel, which knows how
// many m-tiles there are, may cut the columns finer; not with a short K, where a tile's start weighs as much as its walk.
constexpr bool may_narrow(int K) { return k_tiles_of(K) >= kNarrowFromK; }
constexpr long long most_tiles(long long m_tiles, int n, int K, int cus) {
    const long long tiles = m_tiles * n;
    return may_narrow(K) && tiles < cus ? cus : tiles;
}

// How an output's N columns are cut into tiles: n tiles of `columns` (a multiple of 8 unless it is all that a tile can hold).
struct ColumnTiles {
    int n, columns;
};
// What the device knows about a product when it chooses them: m-tiles, slots that have rows, all rows, and the fewest tiles.
struct Product {
    int m_tiles, slots, rows, rows_per_column;  // weight rows per output column: 2 for SwiGLU, else 1
    int N, k_tiles;    // N a multiple of 8
    bool whole_lines;  // K a multiple of kTileK
    int max_tiles;     // that the launch has workgroups for
    float per_cus;     // 1 / CUs
    ColumnTiles fewest;
};
// To whole numbers, of values from 0 to 2^31.
constexpr float down(float v) { return (float)(int)v; }
constexpr float up(float v) { return down(v) + (down(v) < v ? 1.0f : 0.0f); }
// Narrower column tiles than a tile can hold, where those leave CUs idle or a last round nearly empty.
// Whether the fewest are kept without weighing up others: the rounds are full as it is (or there are no rows), of one round less is
// expected; or K is short.  (12 K tiles: 19.0 -> 19.5 us.  The limits of 24 and 32 are older than the price of a tile's start in
// weigh_columns() and no longer needed for its sake: without them products of 17 to 31 K tiles are 1.06 to 1.36 times as fast in the mean,
// weights from HBM, and 0.97 to 1.12 from the Infinity Cache.)
constexpr bool fewest_stay(const Product& p) {
    const float rounds = p.m_tiles * p.fewest.n * p.per_cus;
    if (rounds * 16.0f >= up(rounds) * (rounds <= 1.0f ? 14.0f : 15.0f)) return true;
    return p.k_tiles < (rounds <= 1.0f ? 32 : p.whole_lines ? 24 : kNarrowFromK);
}
// Tiles of 8 * `eighths` columns, `n` of them, and what they cost; whole numbers all but the cost.
struct ColumnChoice {
    float eighths, n, cost;
};
// `more` column tiles (0 .. 63) than the fewest; the least cost is taken.  Per K tile a CU takes as long as it takes to request the lines of
// the tile's weight rows and token rows, and kFixedLines more: MFMAs, barrier and latency of a K tile do not shrink with its
// columns.  A round of the chip's CUs is bound by HBM where that delivers the weight rows later, a slot's m-tiles sharing theirs
// (kHbm: its time for as many lines as all CUs request).  A tile's start costs kStart lines, which finding out what to take (0.3 us) is part
// of.  Tiles of fewer than 32 columns (an MFMA block's), and what is not 4 % better than the fewest, are not taken.
// Measured against the fewest on 2630 products of 23 to 300 rows per slot whose rounds are not full, weights from HBM: 1.169 times as fast in the
// mean, 1.3 % of them slower by more than 2 %, the worst 0.91 (without the fixed part, with 1.7 for kHbm and as narrow as 8 columns:
// 1.149, 3.3 %, 0.68: 31 slots of 25 rows, N 1472, K 5952, 103 us with 128 columns, 149 with 40, 93 as chosen now).  With
// the weights in the Infinity Cache 1.094, 10.7 % and 0.90 (1.072, 16.9 %, 0.68).  kFixedLines 64 to 128, kHbm 1.3 to 1.5 and kStart 2500
// to 5000 are within 0.3 % of each other.
// `rcp` is the reciprocal.
template <class Rcp>
constexpr ColumnChoice weigh_columns(const Product& p, int more, Rcp rcp) {
    constexpr float kFixedLines = 96.0f, kHbm = 1.5f, kStart = 5000.0f, kKeep = 0.96f, kLeastEighths = 4.0f;
    constexpr float kDown = 0.999999f;  // quotients that are whole numbers stay those when rounded up
    const float all = p.N * 0.125f;
    const float eighths = more == 0 ? p.fewest.columns * 0.125f : up(all * rcp((float)(p.fewest.n + more)) * kDown);
    const float n = up(all * rcp(eighths) * kDown);
    const float per_m_tile = rcp((float)p.m_tiles), rounds = p.m_tiles * n * p.per_cus;
    const float whole = down(rounds), begun = up(rounds);
    const float weights = p.rows_per_column * 8 * eighths;              // lines per K tile
    const float per_cu = weights + p.rows * per_m_tile + kFixedLines;
    const float from_hbm = kHbm * weights * p.slots * per_m_tile, last_hbm = from_hbm * (rounds - whole);
    const float walk = whole * (per_cu > from_hbm ? per_cu : from_hbm) + (begun - whole) * (per_cu > last_hbm ? per_cu : last_hbm);
    const float cost = walk * p.k_tiles + kStart * begun;
    if (more == 0) return ColumnChoice{eighths, n, cost * kKeep};
    return ColumnChoice{eighths, n, p.m_tiles * n > p.max_tiles || eighths < kLeastEighths ? 3.0e38f : cost};
}
// The choice as whole numbers: n may be one off in floating point.
constexpr ColumnTiles column_tiles(const Product& p, int eighths, int n) {
    const int columns = 8 * eighths;
    if (n * columns < p.N) ++n;
    else if ((n - 1) * columns >= p.N) --n;
    return p.m_tiles * n > p.max_tiles ? p.fewest : ColumnTiles{n, columns};
}

}  // namespace mid
}  // namespace emoe
