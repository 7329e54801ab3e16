"""The output of an fp32 layer does not depend on which slots its experts lie in: bit for bit the same."""
import pytest
import torch

import paper_2503_06823_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,f,E,k,act", [(64, 128, 256, 8, 2, "swiglu"), (300, 264, 1032, 16, 3, "relu"),
                                           (200, 768, 520, 12, 1, "swiglu")])
def test_output_does_not_depend_on_the_slots(gpu_device, T, d, f, E, k, act):
    g = torch.Generator(device="cuda").manual_seed(11)

    def normal(shape, std):
        return torch.empty(shape, device="cuda").normal_(0.0, std, generator=g)

    x, w_gate = normal((T, d), 1.0), normal((E, d), d ** -0.5)
    w1, w3, w2 = normal((E, f, d), d ** -0.5), normal((E, f, d), d ** -0.5), normal((E, d, f), f ** -0.5)
    desc = P.make_desc(T, d, f, E, k, E, "f32", act)
    outputs = []
    for slot_of_expert in (torch.arange(E, device="cuda"), torch.arange(E, device="cuda").flip(0),
                           torch.randperm(E, generator=g, device="cuda")):
        expert_of_slot = slot_of_expert.argsort()
        b = P.LayerBuffers.allocate(desc, "cuda:0")
        P.layer_forward(b, x, w_gate, None, slot_of_expert.to(torch.int32), w1[expert_of_slot].contiguous(),
                        w3[expert_of_slot].contiguous() if act == "swiglu" else None, w2[expert_of_slot].contiguous(),
                        one_call=True)
        torch.cuda.synchronize()
        outputs.append((b.topk_expert, b.topk_weight, b.out))
    for other in outputs[1:]:
        for a, b in zip(outputs[0], other):
            assert torch.equal(a, b)
