// mid_work.h for the host, behind C names.
#include "mid_work.h"

using namespace emoe::mid;

extern "C" {
int cut_sharers(int tiles, int kt, int G) { return make_cut(tiles, kt, G).sharers; }
unsigned cut_share_begin(int tiles, int kt, int G, int g) { return share_begin(make_cut(tiles, kt, G), g); }
int cut_tile_of_boundary(int tiles, int kt, int G, int b) { return tile_of_boundary(make_cut(tiles, kt, G), kt, b); }
}
