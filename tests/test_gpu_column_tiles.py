"""Layers on tiles of 64 and 128 token rows whose tiles do not fill the chip's rounds, so that the kernel cuts the columns into narrower
tiles: SwiGLU and ReLU, extents that are no multiple of a tile, slots without rows, launches of a workgroup per tile and
persistent ones (K of 64 K tiles and more, not cut along K), the sort inside the first product, rows stored through the permutation.
Which products take narrower tiles is said for each layer, and checked by the rule itself without a GPU in test_mid_work.py."""
import numpy as np
import pytest
import torch

import emoe_inputs as gen
import oracle
import paper_2503_06823_amd as P
from gpu_util import MID, DeviceLayer, check_ffn_rows, check_outputs, check_routing_and_permutation, desc_of, ffn_path
from mid_work import product_tiles

pytestmark = pytest.mark.gpu


def cfg(name, index, **kw):
    return gen.LayerConfig(name=name, index=index, dtype="bf16", **kw)


CASES = [
    cfg("rows128_empty_slots_ktail", 460, T=357, d_model=1288, d_ff=2824, E=24, k=3, R=11, S=20, zipf_s=1.1, act="swiglu"),
    cfg("rows128_whole_lines", 461, T=250, d_model=1152, d_ff=2944, E=8, k=2, R=6, act="swiglu"),
    cfg("rows64_top1_relu", 462, T=500, d_model=1160, d_ff=2056, E=16, k=1, R=8, act="relu"),
    cfg("rows128_top1_swiglu", 467, T=500, d_model=2120, d_ff=2056, E=16, k=1, R=8, act="swiglu"),
    cfg("rows64_swiglu", 463, T=120, d_model=1288, d_ff=4616, E=8, k=2, R=8, act="swiglu"),
    cfg("rows64_relu_top1", 464, T=330, d_model=2120, d_ff=2056, E=16, k=1, R=11, zipf_s=1.1, act="relu"),
    cfg("persistent_whole_tiles_ktail", 465, T=200, d_model=2056, d_ff=4104, E=8, k=2, R=7, act="swiglu"),
    cfg("persistent_whole_tiles_relu", 466, T=160, d_model=2120, d_ff=4160, E=8, k=2, R=8, act="relu"),
    cfg("persistent_swiglu", 468, T=160, d_model=4104, d_ff=2312, E=8, k=2, R=8, act="swiglu"),
]
# token rows, weight rows of a tile and whether the launch is a persistent one, of the products that take narrower column tiles
NARROWER = {
    "rows128_empty_slots_ktail": [(128, 256, False), (128, 128, False)], "rows128_whole_lines": [None, (64, 128, False)],
    "rows64_top1_relu": [None, (64, 128, False)], "rows128_top1_swiglu": [(128, 128, False), (64, 128, False)],
    "rows64_swiglu": [(64, 256, False), (64, 128, True)], "rows64_relu_top1": [(64, 128, False), None],
    "persistent_whole_tiles_ktail": [None, (128, 128, True)], "persistent_whole_tiles_relu": [(64, 128, False), (64, 128, True)],
    "persistent_swiglu": [(128, 128, True), (64, 128, False)],
}


def narrower(c, slot_counts):
    """As NARROWER, by the rule."""
    found = []
    for swiglu, columns, inputs in ((c.act == "swiglu", c.d_ff, c.d_model), (False, c.d_model, c.d_ff)):
        t = product_tiles(swiglu, slot_counts, columns, inputs)
        assert not t.cut
        found.append((t.rows, t.weight_rows, t.persist) if t.columns < t.widest else None)
    return found


@pytest.mark.parametrize("c", CASES, ids=lambda c: c.name)
def test_layer_matches_oracle(gpu_device, c):
    assert ffn_path(desc_of(c)) == MID
    inp = gen.make_layer_inputs(c, shuffle_slots=True)
    ref = oracle.layer_forward(inp)
    assert narrower(c, ref.permutation.slot_counts) == NARROWER[c.name]
    dl = DeviceLayer(inp)
    dl.forward()
    torch.cuda.synchronize()
    check_routing_and_permutation(dl, ref)
    check_outputs(dl, ref)
    check_ffn_rows(dl, ref.permutation, np.arange(c.T * c.k))
    dl.check_gather_path_is_identical()
    # called as a whole: the first product sorts, and with one expert per token the second stores its rows through the permutation
    b = dl.buf
    separate = {n: getattr(b, n).clone() for n in ("perm", "inv_perm", "slot_offsets", "out")}
    for name in separate:
        getattr(b, name).fill_(-9)
    P.layer_forward(b, dl.x, dl.w_gate, dl.gate_bias, dl.slot_of_expert, dl.w1, dl.w3, dl.w2, one_call=True)
    torch.cuda.synchronize()
    for name, value in separate.items():
        assert torch.equal(getattr(b, name), value), name
