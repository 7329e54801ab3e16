"""bf16 layers of few rows per slot whose weight rows are not whole 128-byte lines, with less and with more than 128 MiB of
weights in the first product: its loads carry the non-temporal hint below and not above in the streaming kernels, and never in
those of up to 16 tokens."""
import numpy as np
import pytest
import torch

import emoe_inputs as gen
import oracle
from gpu_util import FEW, STREAM, DeviceLayer, check_ffn_rows, check_outputs, check_routing_and_permutation, desc_of, ffn_kernels

pytestmark = pytest.mark.gpu


def cfg(name, index, **kw):
    return gen.LayerConfig(name=name, index=index, E=2, k=1, R=2, dtype="bf16", **kw)


CASES = [
    cfg("first_product_64_MiB", 380, T=5, d_model=4104, d_ff=4104, act="relu"),
    cfg("first_product_128_MiB_relu", 381, T=9, d_model=4104, d_ff=8200, act="relu"),
    cfg("first_product_128_MiB_swiglu", 382, T=40, d_model=4104, d_ff=4104, act="swiglu"),
    cfg("first_product_64_MiB_streamed", 383, T=20, d_model=4104, d_ff=4104, act="relu"),
    cfg("first_product_128_MiB_relu_streamed", 384, T=24, d_model=4104, d_ff=8200, act="relu"),
]


@pytest.mark.parametrize("c", CASES, ids=lambda c: c.name)
def test_layer_matches_oracle(gpu_device, c):
    inp = gen.make_layer_inputs(c)
    ref = oracle.layer_forward(inp)
    dl = DeviceLayer(inp)
    assert ffn_kernels(desc_of(c)) == (FEW if c.T <= 16 else STREAM)
    dl.forward()
    torch.cuda.synchronize()
    check_routing_and_permutation(dl, ref)
    check_outputs(dl, ref)
    check_ffn_rows(dl, ref.permutation, np.arange(c.T * c.k))
    dl.check_gather_path_is_identical()
