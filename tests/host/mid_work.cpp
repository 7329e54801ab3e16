// mid_work.h for the host, behind C names.
#include "mid_work.h"

#include <cmath>
#include <cstdint>

using namespace emoe::mid;

extern "C" {
int cut_sharers(int tiles, int kt, int G) { return make_cut(tiles, kt, G).sharers; }
unsigned cut_share_begin(int tiles, int kt, int G, int g) { return share_begin(make_cut(tiles, kt, G), g); }
// The column tiles of a product whose slots hold `counts` rows (S of them), on a chip of `cus` CUs, the reciprocal off by `ulps` of its
// last places.  out: the fewest tiles' number and width, the chosen ones', whether the tiles are cut along K, token rows and weight
// rows of a tile, whether the launch is a persistent one.
void product_tiles(bool swiglu, const int* counts, int S, int N, int K, int cus, int ulps, int* out) {
    int rows = 0, m_tiles = 0, slots = 0;
    for (int s = 0; s < S; ++s) rows += counts[s];
    const Arrangement tile = arrangement(swiglu, rows, S, N, K, cus);
    for (int s = 0; s < S; ++s) {
        m_tiles += (counts[s] + tile.rows - 1) / tile.rows;
        slots += counts[s] > 0;
    }
    const int widest = swiglu ? tile.weight_rows / 2 : tile.weight_rows;
    const ColumnTiles fewest{(N + widest - 1) / widest, widest};
    const int max_tiles = tile.persist ? INT32_MAX : most_tiles(most_m_tiles(rows, S, tile.rows), fewest.n, K, cus);
    const bool cut = tile.persist && make_cut(m_tiles * fewest.n, k_tiles_of(K), cus).sharers > 0;
    const Product p{m_tiles, slots, rows, swiglu ? 2 : 1, N, k_tiles_of(K), K % kTileK == 0, max_tiles, 1.0f / cus, fewest};
    ColumnTiles chosen = fewest;
    if (!cut && (tile.persist || may_narrow(K)) && !fewest_stay(p)) {
        auto rcp = [&](float v) {
            float r = 1.0f / v;
            for (int i = 0; i < ulps; ++i) r = std::nextafter(r, 2.0f);
            for (int i = 0; i > ulps; --i) r = std::nextafter(r, 0.0f);
            return r;
        };
        ColumnChoice best = weigh_columns(p, 0, rcp);
        for (int more = 1; more < 64; ++more) {
            const ColumnChoice c = weigh_columns(p, more, rcp);
            if (c.cost < best.cost) best = c;
        }
        chosen = column_tiles(p, (int)best.eighths, (int)best.n);
    }
    const int all[9] = {fewest.n, fewest.columns, chosen.n, chosen.columns, cut, tile.rows, tile.weight_rows, tile.persist, m_tiles};
    for (int i = 0; i < 9; ++i) out[i] = all[i];
}
int cut_first_tile(int tiles, int kt, int G, int g) { return first_tile(make_cut(tiles, kt, G), kt, g); }
void cut_pieces(int tiles, int kt, int G, int tile, int* out) {
    const Pieces p = pieces_of(make_cut(tiles, kt, G), tiles, kt, tile);
    out[0] = p.first;
    out[1] = p.end;
}
}
