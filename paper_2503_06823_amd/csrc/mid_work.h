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
// The tile that boundary b between shares b - 1 and b cuts, if this is the first boundary inside it (the one that sees to the
// adding of its pieces), else -1.  The pieces: shares b - 1, b, ... as long as they begin before the tile's end.
constexpr int tile_of_boundary(Cut cut, int kt, int b) {
    if (b >= cut.sharers) return -1;  // nothing was cut, or no share begins here
    const unsigned at = share_begin(cut, b);
    const int tile = (int)(at / (unsigned)kt);
    const unsigned tile_begin = (unsigned)tile * (unsigned)kt;
    return at != tile_begin && share_begin(cut, b - 1) <= tile_begin ? tile : -1;
}

}  // namespace mid
}  // namespace emoe
