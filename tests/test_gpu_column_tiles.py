"""Layers on tiles of 64 and 128 token rows whose tiles do not fill the chip's rounds, so that the kernel cuts the columns into narrower
tiles: SwiGLU and ReLU, extents that are no multiple of a tile, slots without rows, launches of a workgroup per tile and
persistent ones (K of 64 K tiles and more, not cut along K), the sort inside the first product, rows stored through the permutation."""
import numpy as np
import pytest
import torch

import emoe_inputs as gen
import oracle
from gpu_util import MID, DeviceLayer, check_ffn_rows, check_outputs, check_routing_and_permutation, desc_of, ffn_path

pytestmark = pytest.mark.gpu


def cfg(name, index, **kw):
    return gen.LayerConfig(name=name, index=index, dtype="bf16", **kw)


CASES = [
    cfg("rows128_empty_slots_ktail", 460, T=357, d_model=1288, d_ff=1544, E=24, k=3, R=11, S=20, zipf_s=1.1, act="swiglu"),
    cfg("rows128_whole_lines", 461, T=250, d_model=1152, d_ff=2944, E=8, k=2, R=6, act="swiglu"),
    cfg("rows128_top1_relu", 462, T=500, d_model=1160, d_ff=1416, E=16, k=1, R=8, act="relu"),
    cfg("rows64_swiglu", 463, T=120, d_model=1288, d_ff=1544, E=8, k=2, R=8, act="swiglu"),
    cfg("rows64_relu_top1", 464, T=330, d_model=1096, d_ff=1176, E=16, k=1, R=11, zipf_s=1.1, act="relu"),
    cfg("persistent_whole_tiles_ktail", 465, T=200, d_model=2056, d_ff=4104, E=8, k=2, R=7, act="swiglu"),
    cfg("persistent_whole_tiles_relu", 466, T=160, d_model=2120, d_ff=4160, E=8, k=2, R=8, act="relu"),
]


@pytest.mark.parametrize("c", CASES, ids=lambda c: c.name)
def test_layer_matches_oracle(gpu_device, c):
    assert ffn_path(desc_of(c)) == MID
    inp = gen.make_layer_inputs(c, shuffle_slots=True)
    ref = oracle.layer_forward(inp)
    dl = DeviceLayer(inp)
    dl.forward()
    torch.cuda.synchronize()
    check_routing_and_permutation(dl, ref)
    check_outputs(dl, ref)
    check_ffn_rows(dl, ref.permutation, np.arange(c.T * c.k))
    dl.check_gather_path_is_identical()
