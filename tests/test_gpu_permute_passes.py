"""The counting sort in one workgroup of one, two and four passes and the first size beyond it, against the oracle's stable
permutation: all 64 slots, one slot, slots without rows, and assignments whose expert is not resident (left out)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2503_06823_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 63, 64, 65, 1023, 1024, 1025, 2047, 2048, 2049, 3073, 4095, 4096, 4097])
@pytest.mark.parametrize("E,S,absent", [(64, 64, 0), (1, 1, 0), (24, 20, 0), (40, 33, 7)])
def test_permutation_is_the_stable_one(gpu_device, T, E, S, absent):
    rng = np.random.default_rng(T * 100 + E)
    d = P.make_desc(T, 8, 8, E, 1, S, "bf16", "relu")
    soe = np.full(E, -1, dtype=np.int32)
    soe[rng.permutation(E)[:S]] = rng.permutation(S)
    soe[rng.permutation(np.flatnonzero(soe >= 0))[:absent]] = -1
    pool = np.arange(E) if absent else np.flatnonzero(soe >= 0)  # with `absent`: some assignments are left out
    pool = pool[: max(1, len(pool) - len(pool) // 4)]            # and some slots receive nothing
    te = rng.choice(pool, size=(T, 1)).astype(np.int32)
    b = P.LayerBuffers.allocate(d, "cuda:0")
    b.perm.fill_(-7)
    P.emoe_permute(d, None, torch.from_numpy(te).cuda(), torch.from_numpy(soe).cuda(), b.slot_counts, b.slot_offsets,
                   b.perm, b.inv_perm, None, b.permute_ws, b.permute_ws.numel())
    torch.cuda.synchronize()
    key = soe[te[:, 0]]
    order = np.argsort(np.where(key < 0, S, key), kind="stable")
    placed = int((key >= 0).sum())
    counts = np.bincount(key[key >= 0], minlength=S)
    inv = np.full(T, -1, dtype=np.int32)
    inv[order[:placed]] = np.arange(placed)
    if not absent:
        pm = oracle.permute(te, soe, S)
        assert np.array_equal(pm.perm, order[:placed]) and np.array_equal(pm.slot_counts, counts)
    assert np.array_equal(b.slot_counts.cpu().numpy(), counts)
    assert np.array_equal(b.slot_offsets.cpu().numpy(), np.concatenate([[0], np.cumsum(counts)]))
    assert np.array_equal(b.perm.cpu().numpy()[:placed], order[:placed])
    assert (b.perm.cpu().numpy()[placed:] == -7).all()
    assert np.array_equal(b.inv_perm.cpu().numpy(), inv)
