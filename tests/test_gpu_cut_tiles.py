"""Tiles of 64 and 128 token rows cut along K and put together again, every row compared: pieces that all lie with one XCD's workgroups,
with several and with all; slots of 1 to 32 rows (one block position of a tile has rows), of one tile and of two, empty slots; two
pieces per tile and twenty; SwiGLU, ReLU and plain products; K with and without a tail."""
import pytest

import paper_2503_06823_amd as P
from gpu_util import MID, check_grouped_ffn, ffn_path
from mid_work import lib, product_tiles

pytestmark = pytest.mark.gpu

# activation, rows per slot, d_model, d_ff, which products are cut, with how many shares the first of them
CASES = [
    ("relu", [25], 256, 8384, (False, True), 32), ("relu", [1, 0, 32, 60], 136, 8392, (False, True), 99),
    ("swiglu", [58, 60], 5616, 1024, (True, False), 256), ("swiglu", [140, 0, 33, 66], 4104, 200, (True, False), 130),
    ("relu", [129, 64, 20], 4160, 328, (True, False), 97), ("relu", [40] * 20, 1024, 8256, (False, True), 256),
    ("swiglu", [70, 90, 128, 96], 264, 8200, (False, True), 193),
]


@pytest.mark.parametrize("case", CASES, ids=str)
def test_every_row(gpu_device, case):
    act, rows, d, f, cut, shares = case
    S, T = len(rows), sum(rows)
    desc = P.make_desc(T, d, f, S, 1, S, "bf16", act)
    assert ffn_path(desc) == MID
    products = [product_tiles(act == "swiglu", rows, f, d), product_tiles(False, rows, d, f)]
    assert tuple(p.cut for p in products) == cut
    first = products[cut.index(True)]
    assert lib().cut_sharers(first.m_tiles * first.fewest, -(-(d if cut[0] else f) // 64), 256) == shares
    check_grouped_ffn(desc, act, rows, d + f, gpu_device)
