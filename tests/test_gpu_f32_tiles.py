"""fp32 layers at the edges of the tiles of their kernels: the FFN's 32 tokens (16 per matrix block) x 64 weight rows
x 32 K elements in three LDS stages, the gate's 16 tokens x 16 experts x 32 K elements split over 8 or 16 wavefronts."""
import numpy as np
import pytest
import torch

import emoe_inputs as gen
import oracle
from gpu_util import DeviceLayer, check_ffn_rows, check_outputs, check_routing_and_permutation

pytestmark = pytest.mark.gpu


def cfg(name, index, **kw):
    base = dict(name=name, index=index, T=64, d_model=128, d_ff=256, E=8, k=2, R=4, dtype="f32", act="swiglu")
    base.update(kw)
    return gen.LayerConfig(**base)


CASES = [
    # rows of the only slot around the token block and the tile; K of fewer tiles than there are stages
    cfg("rows_1", 300, T=1, d_model=8, d_ff=8, E=1, k=1, R=1),
    cfg("rows_16", 301, T=16, d_model=24, d_ff=40, E=1, k=1, R=1),
    cfg("rows_17", 302, T=17, d_model=32, d_ff=64, E=1, k=1, R=1, act="relu"),
    cfg("rows_32", 303, T=32, d_model=64, d_ff=72, E=1, k=1, R=1),
    cfg("rows_33", 304, T=33, d_model=72, d_ff=56, E=1, k=1, R=1, act="relu"),
    # K of exactly the stages, one more, with a tail; N of one tile and a tail
    cfg("k_96_104", 305, T=90, d_model=96, d_ff=104, E=4, k=2, R=3, S=4),
    cfg("k_128_136", 306, T=90, d_model=136, d_ff=128, E=4, k=2, R=3, S=4, act="relu"),
    # runs of tiles on every XCD, some slots empty, the sixteen-wavefront gate with a d_model of no whole piece
    cfg("many_tiles", 307, T=700, d_model=264, d_ff=1032, E=64, k=3, R=20, S=24, zipf_s=1.1),
    # expert counts around the blocks of the gate, token counts around its 16
    cfg("experts_17", 308, T=31, d_model=40, d_ff=64, E=17, k=2, R=9),
    cfg("experts_33", 309, T=49, d_model=520, d_ff=64, E=33, k=5, R=17),
    cfg("experts_49_long_rows", 310, T=260, d_model=1536, d_ff=64, E=49, k=2, R=25),
    cfg("experts_64_few_tokens", 311, T=5, d_model=1544, d_ff=64, E=64, k=8, R=64),
    cfg("experts_9_many_tokens", 312, T=1025, d_model=128, d_ff=64, E=9, k=2, R=5),
    cfg("experts_5_many_tokens", 313, T=4097, d_model=64, d_ff=64, E=5, k=1, R=3),
]


@pytest.mark.parametrize("c", CASES, ids=lambda c: c.name)
def test_f32_layer_matches_oracle(gpu_device, c):
    inp = gen.make_layer_inputs(c, shuffle_slots=c.slots > 1)
    ref = oracle.layer_forward(inp)
    dl = DeviceLayer(inp)
    dl.forward()
    torch.cuda.synchronize()
    check_routing_and_permutation(dl, ref)
    check_outputs(dl, ref)
    check_ffn_rows(dl, ref.permutation, np.arange(c.T * c.k))
    dl.check_gather_path_is_identical()
