"""How products on tiles of 64 and 128 token rows are divided.  Tiles cut along K, against whole-number arithmetic of any length: which
products are cut, where the shares begin, and which pieces the second kernel adds; K from one K tile to the longest that an
accepted layer can have.  Column tiles: whatever is chosen covers the columns and fits the tile and the launch."""
import ctypes
import random

import numpy as np
import pytest

import emoe_inputs as gen
import oracle

from mid_work import lib, product_tiles
from test_ffn_path import sorts
from test_gpu_column_tiles import CASES, NARROWER, narrower

LONGEST_K = 1 << 22  # K tiles: d_model * d_ff < 2^31 and 8 columns at least


def reference(tiles, kt, G):
    """sharers, and the first unit of every share with the end of the last: none if the tiles stay whole"""
    if tiles == 0 or tiles >= G:
        return 0, []
    units = tiles * kt
    p = min(units // 8, G)
    if p <= tiles or kt - -(-units // p) < 48:
        return 0, []
    return p, [units * g // p for g in range(p + 1)]


def cases():
    rng = random.Random(20250309)
    yield from [(1, 1, 256), (0, 64, 256), (64, 224, 256), (191, 224, 256), (192, 224, 256), (204, 224, 256), (255, 1 << 14, 256),
                (255, (1 << 14) + 1, 256), (2, (1 << 14) + 1, 256), (255, LONGEST_K, 256), (1, LONGEST_K, 256), (3, 70, 4), (1, 4000, 1)]
    for _ in range(400):
        yield rng.randrange(1, 256), int(2 ** rng.uniform(4, 22)), rng.choice([256, 256, 248, 64, 7])


@pytest.mark.parametrize("long_k", [False, True])
def test_cut_is_exact(long_k):
    seen = 0
    for tiles, kt, G in cases():
        if (kt > 1 << 14) != long_k:
            continue
        sharers, begins = reference(tiles, kt, G)
        assert lib().cut_sharers(tiles, kt, G) == sharers, (tiles, kt, G)
        assert [lib().cut_share_begin(tiles, kt, G, g) for g in range(sharers + 1 if sharers else 0)] == begins, (tiles, kt, G)
        for tile in range(tiles if sharers else 0):  # the shares that hold a part of it
            pieces = (ctypes.c_int * 2)()
            lib().cut_pieces(tiles, kt, G, tile, pieces)
            assert list(range(*pieces)) == [g for g in range(sharers) if begins[g] < (tile + 1) * kt and begins[g + 1] > tile * kt], (tiles, kt, G, tile)
        for first in range(G if sharers else 0):  # a tile begins in one share, and no share holds the beginnings of two
            tile, after = (lib().cut_first_tile(tiles, kt, G, g) for g in (first, first + 1))
            assert tile <= after <= tile + 1 and (after == tile or begins[first] <= tile * kt < begins[first + 1])
        assert not sharers or (lib().cut_first_tile(tiles, kt, G, 0), lib().cut_first_tile(tiles, kt, G, G)) == (0, tiles)
        seen += sharers > 0
    assert seen > 50


def test_column_tiles_cover_the_columns():
    rng = random.Random(20250310)
    narrowed = 0
    for i in range(6000):
        S = int(2 ** rng.uniform(0, 6.001))
        counts = [int(2 ** rng.uniform(0, 8.3)) if rng.random() < 0.9 else 0 for _ in range(S)]
        counts[rng.randrange(S)] += 1
        N, K = (8 * max(1, int(2 ** rng.uniform(3, 15 if i % 10 else 21) / 8)) for _ in range(2))
        if N * K >= 1 << 31:
            continue
        swiglu, cus = rng.random() < 0.5, rng.choice([256, 256, 304, 60])
        for ulps in (-2, 0, 2):  # the device's reciprocal is off by one unit in the last place
            t = product_tiles(swiglu, counts, N, K, cus, ulps)
            assert t.columns % 8 == 0 and 8 <= t.columns <= t.widest and (t.n - 1) * t.columns < N <= t.n * t.columns, (counts, N, K, swiglu, t)
            if not t.persist:  # as many workgroups as the launch has: every slot adds at most one m-tile that is not full
                m_tiles = sum(counts) // t.rows + min(S, sum(counts))
                assert t.m_tiles * t.n <= max(m_tiles * t.fewest, cus if K > 16 * 64 else 0)
        narrowed += t.columns < t.widest
    assert narrowed > 300


# SwiGLU, rows, slots (even ones), outputs, inputs, columns of a tile.  us, weights from HBM: as wide as a tile can hold; narrower than the
# columns given here, which was slower; and with the columns given here, where these are not the widest
SLOWER_BELOW = [
    (True, 816, 27, 896, 4736, 56),    # 88.4, 104.3 with 32, 83.7
    (True, 180, 7, 3456, 5568, 48),    # 101.1, 117.9 with 32, 91.6
    (True, 533, 21, 800, 5120, 40),    # 94.5, 104.2 with 24, 79.9
    (True, 1222, 8, 256, 2048, 32),    # 18.1, 19.4 with 16, 18.1
    (False, 244, 9, 5248, 4976, 96),   # 128.5, 138.8 with 64, 117.2
    (True, 544, 3, 2712, 1648, 64), (False, 563, 3, 5520, 2592, 128), (False, 473, 2, 4352, 2560, 128),  # 41.1, 47.3; 57.8, 65.5; 37.5, 45.0
    (False, 660, 3, 2872, 1936, 128), (False, 2685, 15, 1088, 1984, 128),                                # 38.3, 44.6; 36.3, 41.3
]
# ... and where tiles of up to so many columns were at least 1.25 times as fast as the widest
FASTER_UP_TO = [(False, 39, 1, 296, 3912, 32), (False, 110, 2, 912, 3080, 32), (False, 188, 5, 1440, 3992, 40), (False, 54, 1, 3024, 3784, 40)]


def even(rows, slots):
    return [rows // slots + (i < rows % slots) for i in range(slots)]


@pytest.mark.parametrize("product", SLOWER_BELOW, ids=str)
def test_columns_are_not_cut_where_that_was_slower(product):
    swiglu, rows, slots, N, K, least = product
    t = product_tiles(swiglu, even(rows, slots), N, K)
    assert not t.cut and t.columns >= least, t


@pytest.mark.parametrize("product", FASTER_UP_TO, ids=str)
def test_columns_are_cut_where_that_was_faster(product):
    swiglu, rows, slots, N, K, most = product
    t = product_tiles(swiglu, even(rows, slots), N, K)
    assert not t.cut and t.columns <= most < t.widest, t


@pytest.mark.parametrize("c", CASES, ids=lambda c: c.name)
def test_layers_that_are_to_take_narrower_tiles_do(c):
    inp = gen.make_layer_inputs(c, shuffle_slots=True)
    counts = oracle.layer_forward(inp, tokens=np.arange(1)).permutation.slot_counts
    assert narrower(c, counts) == NARROWER[c.name]


def test_layers_that_sort_in_a_product_of_narrower_tiles():
    found = {c.name for c in CASES if NARROWER[c.name][0] and sorts(c.T, c.d_model, c.d_ff, c.E, c.k, c.slots, c.dtype, c.act)}
    assert found == {"rows128_top1_swiglu", "rows64_swiglu", "rows64_relu_top1", "persistent_whole_tiles_relu", "persistent_swiglu"}
