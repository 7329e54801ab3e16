"""How tiles of 64 and 128 token rows are cut along K, against whole-number arithmetic of any length: which products are cut, where the
shares begin, and which pieces the second kernel adds; K from one K tile to the longest that an accepted layer can have."""
import random

import pytest

from mid_work import lib

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
        # every tile that a boundary falls into has exactly one boundary that sees to it: the first, whose left share holds its start
        owner = {}
        for b in range(1, G):
            tile = lib().cut_tile_of_boundary(tiles, kt, G, b)
            if tile >= 0:
                assert tile not in owner
                owner[tile] = b
        cut_at = [x for x in begins[1:-1] if x % kt]
        assert set(owner) == {x // kt for x in cut_at}, (tiles, kt, G)
        for tile, b in owner.items():
            assert begins[b - 1] <= tile * kt < begins[b] < (tile + 1) * kt
        seen += sharers > 0
    assert seen > 50
