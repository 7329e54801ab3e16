"""Layers of so many 256-row tiles that every workgroup of the persistent launch walks several: the operand stream that runs
on from one output tile to the next, its stores that are still on their way, tiles of 0 to 8 row blocks per wavefront
one after the other, and the tiles at the end that are cut along K; SwiGLU and ReLU, K with and without a tail, slots of one
and of many tiles, and (k = 1) rows stored through the permutation.  Compared with the oracle on a row of every 16-row
block of every slot, over all columns.  And layers of few such tiles, most of them cut along K."""
import numpy as np
import pytest
import torch

import emoe_inputs as gen
import oracle
import paper_2503_06823_amd as P
from gpu_util import (TILED, DeviceLayer, check_ffn_rows, check_outputs, check_routing_and_permutation, desc_of, ffn_path,
                      stratified_rows)

pytestmark = pytest.mark.gpu

WORKGROUPS = 256  # of the persistent launch


def cfg(name, index, **kw):
    return gen.LayerConfig(name=name, index=index, dtype="bf16", **kw)


CASES = [
    cfg("swiglu_ktail", 420, T=14000, d_model=1032, d_ff=2056, E=8, k=2, R=5, S=6, zipf_s=1.1, act="swiglu"),
    cfg("relu_ktail_top1", 421, T=30000, d_model=1032, d_ff=1160, E=8, k=1, R=6, act="relu"),
    cfg("swiglu_whole_lines_top1", 422, T=28000, d_model=1280, d_ff=1024, E=8, k=1, R=5, zipf_s=1.1, act="swiglu"),
    cfg("relu_whole_lines", 423, T=15000, d_model=1152, d_ff=1344, E=6, k=2, R=4, act="relu"),
    # slots of one m-tile (without the tail: their weights carry the non-temporal hint) beside slots of many
    cfg("many_slots_ktail", 424, T=12000, d_model=776, d_ff=1160, E=64, k=2, R=64, zipf_s=0.7, act="swiglu"),
    cfg("many_slots_whole_lines_top1", 425, T=30000, d_model=1024, d_ff=832, E=64, k=1, R=50, S=60, zipf_s=1.1, act="relu"),
]


@pytest.mark.parametrize("c", CASES, ids=lambda c: c.name)
def test_layer_of_many_tiles(gpu_device, c):
    assert ffn_path(desc_of(c)) == TILED
    inp = gen.make_layer_inputs(c, shuffle_slots=True)
    tokens = np.sort(np.random.default_rng(c.seed).choice(c.T, 24, replace=False))
    ref = oracle.layer_forward(inp, tokens=tokens)
    counts = ref.permutation.slot_counts
    m_tiles = int(((counts + 255) // 256).sum())
    for columns, tile in ((c.d_ff, 128 if c.act == "swiglu" else 256), (c.d_model, 256)):
        tiles = m_tiles * (-(-columns // tile))
        assert tiles > 2 * WORKGROUPS and tiles % WORKGROUPS, f"{tiles} tiles"
    print(f"{c.name}: {m_tiles} m-tiles, rows per slot {counts.min()} to {counts.max()}", flush=True)
    dl = DeviceLayer(inp)
    dl.forward()
    torch.cuda.synchronize()
    check_routing_and_permutation(dl, ref)
    check_outputs(dl, ref)
    check_ffn_rows(dl, ref.permutation, stratified_rows(ref.permutation.slot_offsets, c.seed))
    dl.check_gather_path_is_identical()
    if c.k > 1:
        return
    b = dl.buf
    separate = b.out.clone()
    b.out.fill_(float("nan"))
    P.emoe_expert_ffn_gather_combine(dl.desc, dl.x, b.perm, b.inv_perm, b.slot_offsets, dl.w1, dl.w3, dl.w2, b.topk_weight,
                                     None, b.out, b.ffn_ws, b.ffn_ws.numel())
    torch.cuda.synchronize()
    assert torch.equal(b.out.view(torch.int16), separate.view(torch.int16))


def _random_cases(n, seed):
    """Seeded random layers with few 256-row tiles, from 301 rows per slot on, one of the two K long in every other one:
    cut along K into up to eight pieces, ragged in both directions, slots without rows."""
    rng = np.random.default_rng(seed)
    cases = []
    for i in range(n):
        act = "relu" if rng.random() < 0.4 else "swiglu"
        E = int(rng.choice([1, 2, 4, 8, 16]))
        R = int(rng.integers(1, E + 1))
        k = int(rng.integers(1, min(R, 4) + 1))
        S = int(rng.integers(R, E + 1))
        T = -(-int(rng.choice([301, 330, 420, 513])) * S // k)
        d_model, d_ff = int(rng.choice([64, 136, 264, 520])), int(rng.choice([64, 72, 200, 512]))
        if i % 4 == 0:
            d_model = int(rng.choice([2048, 4104]))
        elif i % 4 == 2:
            d_ff = int(rng.choice([2056, 4096]))
        cases.append(cfg(f"random{i}_{act}_T{T}_d{d_model}_f{d_ff}_E{E}_k{k}_R{R}_S{S}", 430 + i, act=act, T=T, d_model=d_model,
                         d_ff=d_ff, E=E, k=k, R=R, S=S, zipf_s=float(rng.choice([0.0, 1.1]))))
    return cases


@pytest.mark.parametrize("c", _random_cases(16, 20250308), ids=lambda c: c.name)
def test_random_layer_of_few_tiles(gpu_device, c):
    assert ffn_path(desc_of(c)) == TILED
    inp = gen.make_layer_inputs(c, shuffle_slots=c.slots > 1)
    tokens = np.sort(np.random.default_rng(c.seed).choice(c.T, min(c.T, 64), replace=False))
    ref = oracle.layer_forward(inp, tokens=tokens)
    dl = DeviceLayer(inp)
    dl.forward()
    torch.cuda.synchronize()
    check_routing_and_permutation(dl, ref)
    check_outputs(dl, ref)
    check_ffn_rows(dl, ref.permutation, stratified_rows(ref.permutation.slot_offsets, c.seed))
    dl.check_gather_path_is_identical()
