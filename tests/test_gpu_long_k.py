"""A second product of more than 2^20 in K, two tiles cut along K into 256 shares and put together again: whole numbers small enough that
fp32 sums are exact in any order, so that every element has to be the rounded exact sum; beside it a length that leaves a K tail."""
import pytest
import torch

import paper_2503_06823_amd as P
from gpu_util import MID, ffn_path
from mid_work import lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("f", [(1 << 20) + 64, (1 << 20) + 72])
def test_cut_along_a_long_k(gpu_device, f):
    T, d, S = 60, 64, 2
    desc = P.make_desc(T, d, f, S, 1, S, "bf16", "relu")
    assert ffn_path(desc) == MID and lib().cut_sharers(S, -(-f // 64), 256) == 256
    g = torch.Generator(device=gpu_device)
    g.manual_seed(f)

    def whole(*shape):  # -1, 0 or 1
        return torch.randint(-1, 2, shape, generator=g, device=gpu_device, dtype=torch.int8).bfloat16()

    x, w1, w2 = whole(T, d), whole(S, f, d), whole(S, d, f)  # h: whole numbers up to 64, exact in bf16
    offsets = torch.tensor([0, 25, T], dtype=torch.int32, device=gpu_device)
    b = P.LayerBuffers.allocate(desc, gpu_device)
    b.y_perm.fill_(float("nan"))
    P.emoe_expert_ffn(desc, x, offsets, w1, None, w2, b.y_perm, b.ffn_ws, b.ffn_ws.numel())
    torch.cuda.synchronize()
    for s, (lo, hi) in enumerate([(0, 25), (25, T)]):
        h = torch.relu(x[lo:hi].float() @ w1[s].float().t())
        y = h @ w2[s].float().t()
        assert float((h @ w2[s].float().abs().t()).max()) < 2 ** 24  # no partial sum is larger: exact in any order
        assert torch.equal(b.y_perm[lo:hi], y.bfloat16())
