"""Logits that are no numbers: every gate kernel ranks a NaN after all numbers (-inf included), the lower expert first among
several, for the routing and for the observed workload alike.  Token and gate rows are small integers, as in test_gpu_ties, so
that all other logits are exact; the NaN and the -inf come with the bias."""
import numpy as np
import pytest
import torch

import oracle
import paper_2503_06823_amd as P
import test_gpu_ties as ties
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

# gate kernel, dtype, T, d_model, E, k, R
CASES = [
    ("wavefront", "bf16", 21, 2048, 8, 3, 6), ("wavefront", "bf16", 256, 2056, 4, 3, 3), ("wavefront", "bf16", 5, 4096, 2, 2, 2),
    ("wavefront", "bf16", 17, 6152, 16, 10, 10), ("matrix", "bf16", 16, 6152, 16, 10, 10), ("wavefront", "bf16", 9, 8192, 11, 5, 5),
    ("matrix", "bf16", 257, 2048, 8, 3, 6), ("matrix", "bf16", 21, 72, 20, 12, 12), ("matrix", "bf16", 5000, 64, 64, 3, 40),
    ("wavefront", "f32", 21, 64, 8, 6, 6), ("wavefront", "f32", 300, 128, 12, 3, 9), ("wavefront", "f32", 21, 4096, 20, 3, 12),
    ("wavefront", "f32", 33, 2048, 64, 40, 40), ("wavefront", "f32", 2100, 64, 4, 3, 3),
    ("matrix", "f32", 21, 72, 20, 12, 12), ("matrix", "f32", 1030, 64, 12, 3, 9), ("matrix", "f32", 4100, 64, 8, 3, 6),
    ("matrix", "f32", 300, 512, 40, 6, 30),
]


def ranked(logits, k):
    """The k best columns of every row: descending, NaN last, the lower column first among equals."""
    key = np.where(np.isnan(logits), 0.0, -logits)
    return np.lexsort((np.broadcast_to(np.arange(logits.shape[1]), logits.shape), key, np.isnan(logits)), axis=1)[:, :k]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "_".join(map(str, c)))
def test_nan_comes_after_all_numbers(gpu_device, case):
    _, dtype, T, d, E, k, R = case
    x, wg, _, soe = ties.tie_inputs(dtype, T, d, E, R, max(2, E // 3), False, seed=T + E)
    resident = np.flatnonzero(soe >= 0)
    bias = np.zeros(E, dtype=np.float32)
    bias[[0, resident[0], resident[R // 2]]] = np.nan
    if R > 2:
        bias[resident[1]] = -np.inf
    with np.errstate(invalid="ignore"):
        logits = oracle.gate_logits(x, wg, None, dtype) + bias
        idx = resident[ranked(logits[:, resident], k)]
        sel = np.take_along_axis(logits, idx, axis=1)
        p = np.exp(sel - sel[:, :1])
        weight = p / p.sum(axis=1, keepdims=True)  # a NaN among the winners makes all of a token's weights NaN
    workload = np.bincount(ranked(logits, k).reshape(-1), minlength=E)

    te = torch.full((T, k), -7, dtype=torch.int32, device="cuda")
    tw = torch.full((T, k), -7.0, device="cuda")
    counts = torch.zeros(E, dtype=torch.int64, device="cuda")
    P.emoe_route_observe(P.make_desc(T, d, 64, E, k, R, dtype, "swiglu"), to_dev(x, dtype), to_dev(wg, dtype),
                         torch.from_numpy(bias).cuda(), torch.from_numpy(soe).cuda(), te, tw, counts)
    torch.cuda.synchronize()
    assert np.array_equal(te.cpu().numpy(), idx)
    assert np.array_equal(counts.cpu().numpy(), workload)
    got = tw.cpu().numpy()
    assert np.array_equal(np.isnan(got), np.isnan(weight))
    assert np.nanmax(np.abs(got - weight), initial=0.0) <= 1e-5
