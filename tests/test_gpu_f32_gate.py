"""The fp32 gate on both sides of the rules that choose its kernel: a wavefront's or four wavefronts' walk per token with all or
four experts' loads at a time, or 16 tokens together on the matrix instructions."""
import pytest
import torch

import emoe_inputs as gen
import oracle
from gpu_util import DeviceLayer, check_routing_and_permutation

pytestmark = pytest.mark.gpu


def cfg(E, d, T, k, zipf=0.0):
    return gen.LayerConfig(name=f"E{E}_d{d}_T{T}", index=400 + E, T=T, d_model=d, d_ff=8, E=E, k=k, R=max(k, E // 2), dtype="f32",
                           act="relu", zipf_s=zipf)


CASES = [cfg(7, 520, 256, 2), cfg(7, 520, 257, 2), cfg(8, 1032, 2049, 1, 1.1), cfg(5, 1032, 4095, 2),
         cfg(9, 264, 256, 3), cfg(9, 264, 257, 3), cfg(16, 2056, 512, 2, 1.1), cfg(13, 1288, 513, 4), cfg(16, 136, 1023, 1),
         cfg(17, 4096, 256, 2), cfg(32, 4104, 255, 6, 1.1), cfg(24, 4096, 257, 3), cfg(32, 5120, 512, 2), cfg(20, 5128, 513, 2),
         cfg(17, 4088, 3, 8), cfg(40, 2048, 256, 2), cfg(33, 2056, 257, 5), cfg(48, 2040, 64, 3, 1.1), cfg(64, 1536, 256, 8),
         cfg(49, 1528, 256, 2)]


@pytest.mark.parametrize("c", CASES, ids=lambda c: c.name)
def test_routing_matches_oracle(gpu_device, c):
    inp = gen.make_layer_inputs(c, shuffle_slots=True)
    ref = oracle.layer_forward(inp, with_ffn=False)
    dl = DeviceLayer(inp)
    dl.forward()
    torch.cuda.synchronize()
    check_routing_and_permutation(dl, ref)
