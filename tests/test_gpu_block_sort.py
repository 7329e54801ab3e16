"""A layer called as a whole, whose first product sorts the assignments itself, against the four calls one by one: the
permutation, the slots' sizes and the results must be the same bits.  Every kernel that sorts, at one assignment, at sizes
around its passes of 256 assignments (four wavefronts) and 512 (eight: layers of up to 16 tokens with long rows and few workgroups),
at 1024 and one past it, with empty slots, popular experts, several tiles and passes per slot, and with fewer than k resident
experts: assignments that appear in no slot, or all in one, which then takes several trips."""
import numpy as np
import pytest
import torch

import emoe_inputs as gen
import paper_2503_06823_amd as P
from gpu_util import DeviceLayer

pytestmark = pytest.mark.gpu

# dtype, T, d_model, d_ff, E, k, R, S, activation, popularity
CASES = [
    ("f32", 1, 64, 96, 1, 1, 1, 1, "relu", 0.0), ("f32", 64, 136, 264, 8, 2, 4, 6, "swiglu", 0.0), ("f32", 255, 72, 64, 64, 4, 60, 64, "swiglu", 1.1),
    ("f32", 1024, 64, 128, 64, 1, 20, 24, "relu", 1.2), ("f32", 1025, 64, 128, 64, 1, 20, 24, "relu", 1.2),
    ("bf16", 1, 264, 2056, 8, 2, 6, 6, "swiglu", 0.0), ("bf16", 16, 2056, 264, 64, 8, 60, 64, "relu", 0.0), ("bf16", 13, 2200, 520, 8, 3, 5, 7, "swiglu", 0.0),
    ("bf16", 16, 2048, 64, 64, 32, 64, 64, "swiglu", 0.0), ("bf16", 16, 2056, 64, 64, 33, 64, 64, "swiglu", 0.0), ("bf16", 16, 2048, 64, 64, 64, 64, 64, "relu", 0.0),
    ("bf16", 15, 264, 72, 64, 17, 60, 64, "swiglu", 0.0), ("bf16", 16, 264, 64, 64, 33, 64, 64, "relu", 0.0), ("bf16", 16, 264, 64, 64, 64, 64, 64, "swiglu", 0.0),
    ("bf16", 16, 2056, 2568, 8, 3, 3, 3, "relu", 0.0), ("bf16", 16, 2056, 2064, 2, 1, 2, 2, "swiglu", 0.0),
    ("bf16", 17, 264, 328, 8, 2, 6, 8, "swiglu", 0.0), ("bf16", 60, 328, 264, 24, 3, 11, 20, "swiglu", 1.2), ("bf16", 128, 264, 328, 64, 8, 60, 64, "relu", 1.1),
    ("bf16", 86, 264, 328, 8, 3, 6, 8, "swiglu", 1.1), ("bf16", 171, 520, 328, 16, 3, 12, 12, "relu", 1.2), ("bf16", 1024, 136, 264, 64, 1, 16, 20, "relu", 1.1),
    ("bf16", 341, 4104, 264, 4, 3, 4, 4, "relu", 0.0), ("bf16", 100, 4104, 200, 2, 1, 2, 2, "relu", 0.0), ("bf16", 200, 1032, 2808, 24, 5, 20, 24, "swiglu", 1.1),
]


def forward(dl, one_call):
    b = dl.buf
    for t in (b.slot_counts, b.slot_offsets, b.perm, b.inv_perm, b.topk_expert):
        t.fill_(-9)
    b.y_perm.fill_(float("nan"))
    b.out.fill_(float("nan"))
    P.layer_forward(b, dl.x, dl.w_gate, dl.gate_bias, dl.slot_of_expert, dl.w1, dl.w3, dl.w2, one_call=one_call)
    torch.cuda.synchronize()
    return {n: getattr(b, n).clone() for n in ("slot_counts", "slot_offsets", "perm", "inv_perm", "topk_expert", "topk_weight", "out")}


@pytest.mark.parametrize("case", CASES, ids=lambda c: "_".join(map(str, c[:9])))
def test_whole_layer_equals_the_four_calls(gpu_device, case):
    dtype, T, d, f, E, k, R, S, act, zipf = case
    c = gen.LayerConfig(name="sort", index=800, T=T, d_model=d, d_ff=f, E=E, k=k, R=R, S=S, act=act, dtype=dtype, zipf_s=zipf)
    dl = DeviceLayer(gen.make_layer_inputs(c, shuffle_slots=True, enforce_margin=k < 16))  # (with many choices every token has a close one)
    one, four = forward(dl, True), forward(dl, False)
    for name, value in four.items():
        assert torch.equal(one[name], value), name
    # fewer than k resident experts: expert 0 fills the places that are left, in no slot if it is not resident itself, else in the same
    if k > 1 and E > 2:
        dl.slot_of_expert.fill_(-1)
        dl.slot_of_expert[E - 1] = S - 1
        one, four = forward(dl, True), forward(dl, False)
        assert (four["inv_perm"] < 0).any()
        for name in ("slot_counts", "slot_offsets", "inv_perm", "topk_expert"):
            assert torch.equal(one[name], four[name]), name
        n = int(four["slot_offsets"][S])
        assert torch.equal(one["perm"][:n], four["perm"][:n])
        dl.slot_of_expert.fill_(-1)
        dl.slot_of_expert[0] = S - 1
        one, four = forward(dl, True), forward(dl, False)
        assert int(four["slot_counts"][S - 1]) == T * k
        for name, value in four.items():
            assert torch.equal(one[name], value), name
