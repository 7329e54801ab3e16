"""bf16 layers at the edges of the rules that choose their path and of the cache hint on their weights: rows that are
not whole 128-byte lines in each path (streamed, tiles of 64, 128 and 256 token rows), small layers of 100 to 300 rows per slot,
and K of fewer K tiles than a tile's loads run ahead."""
import numpy as np
import pytest
import torch

import emoe_inputs as gen
import oracle
from gpu_util import (MID, STREAM, TILED, DeviceLayer, check_ffn_rows, check_outputs, check_routing_and_permutation, desc_of,
                      ffn_path)

pytestmark = pytest.mark.gpu


def cfg(name, index, **kw):
    base = dict(name=name, index=index, T=64, d_model=128, d_ff=256, E=8, k=2, R=4, dtype="bf16", act="swiglu")
    base.update(kw)
    return gen.LayerConfig(**base)


CASES = [
    # K of one to six tiles, with and without a tail: the loads run two to five tiles ahead, a quarter of a tile at a time
    cfg("k_8", 340, T=23, d_model=8, d_ff=8, E=1, k=1, R=1),
    cfg("k_64_128", 341, T=32, d_model=64, d_ff=128, E=1, k=1, R=1, act="relu"),
    cfg("k_192_200", 345, T=120, d_model=192, d_ff=200, E=8, k=2, R=5, S=7),
    cfg("k_256_264", 346, T=120, d_model=264, d_ff=256, E=8, k=3, R=5, S=6, act="relu"),
    cfg("k_320_384", 347, T=300, d_model=320, d_ff=384, E=16, k=2, R=12, zipf_s=1.1),
    # small layers on both sides of 300 rows per slot
    cfg("small_101_rows", 351, T=202, d_model=520, d_ff=640, E=2, k=1, R=2),
    cfg("small_300_rows", 356, T=600, d_model=512, d_ff=1408, E=2, k=1, R=2),
    cfg("small_301_rows", 357, T=602, d_model=256, d_ff=648, E=2, k=1, R=2),
    # rows that are not whole lines: streamed (one slot above a pass, K tail of a line and of less), 128- and 256-row tiles
    cfg("stream_split_lines", 352, T=60, d_model=200, d_ff=392, E=4, k=1, R=4, zipf_s=1.1),
    cfg("stream_whole_lines_tail", 353, T=40, d_model=192, d_ff=320, E=4, k=2, R=4),
    cfg("mid_split_lines", 354, T=1200, d_model=520, d_ff=2056, E=16, k=1, R=16),
    cfg("tiled_split_lines", 355, T=2600, d_model=1032, d_ff=2056, E=8, k=1, R=8),
]

PATHS = {"k_8": MID, "k_64_128": MID, "k_192_200": MID, "k_256_264": MID, "k_320_384": MID, "small_101_rows": MID,
         "small_300_rows": MID, "small_301_rows": TILED, "stream_split_lines": STREAM, "stream_whole_lines_tail": STREAM,
         "mid_split_lines": MID, "tiled_split_lines": TILED}


@pytest.mark.parametrize("c", CASES, ids=lambda c: c.name)
def test_layer_matches_oracle(gpu_device, c):
    assert ffn_path(desc_of(c)) == PATHS[c.name]
    inp = gen.make_layer_inputs(c, shuffle_slots=c.slots > 1)
    ref = oracle.layer_forward(inp)
    dl = DeviceLayer(inp)
    dl.forward()
    torch.cuda.synchronize()
    check_routing_and_permutation(dl, ref)
    check_outputs(dl, ref)
    check_ffn_rows(dl, ref.permutation, np.arange(c.T * c.k))
    dl.check_gather_path_is_identical()
