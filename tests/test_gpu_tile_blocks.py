"""256-row tiles by the number of their 16-row blocks that hold rows: every number that the K loop is compiled for (0 to 8 for each
of the two rows of wavefronts), with a last block that is full, half full and of one row, beside slots of two, three and more
than eight tiles; K of two K tiles (an item requests the next one's operands from its start), of several, and with a tail."""
import pytest
import torch

import paper_2503_06823_amd as P
from gpu_util import TILED, ffn_path

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("act", ["swiglu", "relu"])
@pytest.mark.parametrize("d,f", [(128, 128), (128, 392), (392, 256)])
@pytest.mark.parametrize("missing", [0, 7, 15])
def test_every_number_of_blocks(gpu_device, act, d, f, missing):
    rows = [16 * b - missing for b in range(1, 17)] + [0, 257, 272, 512 - missing, 515, 2049 + missing, 7000]
    S, T = len(rows), sum(rows)
    desc = P.make_desc(T, d, f, S, 1, S, "bf16", act)
    assert ffn_path(desc) == TILED
    g = torch.Generator(device=gpu_device)
    g.manual_seed(100 * missing + d + f)

    def normal(shape, std):
        return torch.empty(shape, dtype=torch.bfloat16, device=gpu_device).normal_(0.0, std, generator=g)

    x, w1, w2 = normal((T, d), 1.0), normal((S, f, d), d ** -0.5), normal((S, d, f), f ** -0.5)
    w3 = normal((S, f, d), d ** -0.5) if act == "swiglu" else None
    perm = torch.randperm(T, generator=g, device=gpu_device).to(torch.int32)
    offsets = torch.tensor([sum(rows[:s]) for s in range(S + 1)], dtype=torch.int32, device=gpu_device)
    b = P.LayerBuffers.allocate(desc, gpu_device)
    b.y_perm.fill_(float("nan"))
    P.emoe_expert_ffn_gather(desc, x, perm, offsets, w1, w3, w2, b.y_perm, b.ffn_ws, b.ffn_ws.numel())
    torch.cuda.synchronize()
    for s in range(S):
        o = int(offsets[s])
        xs = x[perm[o:o + rows[s]].long()].float()
        h = xs @ w1[s].float().t()
        h = torch.nn.functional.silu(h) * (xs @ w3[s].float().t()) if act == "swiglu" else torch.relu(h)
        h = h.bfloat16().float()
        y = h @ w2[s].float().t()
        # h may round to the other neighbour (2^-8 of each), y is rounded once (2^-9), sums in fp32
        bound = 2.0 ** -8 * (h.abs() @ w2[s].float().abs().t()) + 2.0 ** -8 * y.abs() + 1e-5
        err = (b.y_perm[o:o + rows[s]].float() - y).abs()
        assert bool((err <= bound).all()), f"slot {s} of {rows[s]} rows: {float((err - bound).max())}"
