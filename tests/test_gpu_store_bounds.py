"""What the 256-row tiles store stays inside the output: every wavefront issues all of a tile's stores and those of rows
and columns that do not exist are dropped by their address.  Memory on both sides of h, y_perm and out, and the rows of
y_perm behind the last grouped row, keep their contents; tiles are ragged in both directions."""
import pytest
import torch

import paper_2503_06823_amd as P

pytestmark = pytest.mark.gpu

TILED_PARTIALS = 256 + (64 << 20)  # what the workspace holds beside h on this path
GUARD = 4096                       # bytes on each side
FILL = 0x5A


def guarded(nbytes):
    """A buffer with guards: (whole, its middle)."""
    whole = torch.full((nbytes + 2 * GUARD,), FILL, dtype=torch.uint8, device="cuda")
    return whole, whole[GUARD:GUARD + nbytes]


def guards_untouched(whole):
    return bool((whole[:GUARD] == FILL).all()) and bool((whole[-GUARD:] == FILL).all())


@pytest.mark.parametrize("T,d,f,S,k,act", [
    (1201, 264, 456, 3, 2, "swiglu"),  # K tails, a last n-tile of 8 and of 72 columns
    (997, 520, 648, 3, 1, "relu"),     # k = 1: also with the rows stored through perm
    (2600, 1032, 2056, 8, 1, "swiglu"),
])
def test_stores_stay_inside_the_output(gpu_device, T, d, f, S, k, act):
    g = torch.Generator(device="cuda").manual_seed(7)
    desc = P.make_desc(T, d, f, S + 1, k, S, "bf16", act)
    A = T * k
    _, ws_bytes = P.emoe_workspace_bytes(desc)
    assert ws_bytes == (A * f * 2 + 255) // 256 * 256 + TILED_PARTIALS, "not the 256-row tiles any more"

    def normal(*shape):
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.05, generator=g)

    x, w1, w3, w2 = normal(T, d), normal(S, f, d), normal(S, f, d) if act == "swiglu" else None, normal(S, d, f)
    # the last expert has no slot: its assignments are left out, and the grouped rows end before row A
    slot_of_expert = torch.tensor([*range(S), -1], dtype=torch.int32, device="cuda")
    topk = torch.stack([torch.randperm(S + 1, generator=g, device="cuda")[:k] for _ in range(T)]).to(torch.int32)
    b = P.LayerBuffers.allocate(desc, "cuda:0")
    P.emoe_permute(desc, x, topk, slot_of_expert, b.slot_counts, b.slot_offsets, b.perm, b.inv_perm, None, b.permute_ws,
                   b.permute_ws.numel())
    placed = int(b.slot_offsets[-1])
    assert 0 < placed < A
    ws_whole, ws = guarded(ws_bytes)
    y_whole, y = guarded(A * d * 2)
    P.emoe_expert_ffn_gather(desc, x, b.perm, b.slot_offsets, w1, w3, w2, y, ws, ws_bytes)
    torch.cuda.synchronize()
    assert guards_untouched(ws_whole) and guards_untouched(y_whole)
    assert bool((y[placed * d * 2:] == FILL).all()), "rows behind the last grouped row"
    assert bool((ws[placed * f * 2:A * f * 2] == FILL).all()), "rows of h behind the last grouped row"
    rows = y.view(torch.bfloat16).view(A, d)[:placed]
    assert torch.isfinite(rows.float()).all() and bool((rows != 0).any(dim=1).all())
    if k > 1:
        return
    out_whole, out = guarded(T * d * 2)
    P.emoe_expert_ffn_gather_combine(desc, x, b.perm, b.inv_perm, b.slot_offsets, w1, w3, w2, b.topk_weight, None,
                                     out, ws, ws_bytes)
    torch.cuda.synchronize()
    assert guards_untouched(ws_whole) and guards_untouched(out_whole)
    got = out.view(torch.int16).view(T, d)
    here = b.perm[:placed].long()
    assert torch.equal(got[here], y.view(torch.int16).view(A, d)[:placed])
    absent = (topk[:, 0] == S).nonzero().flatten()
    assert bool((out.view(T, d * 2)[absent] == FILL).all()), "rows of tokens whose expert has no slot"
