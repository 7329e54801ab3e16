"""The bf16 gate where its matrix-core kernel cuts: 16 or 32 tokens per workgroup (32 from more than 16 per CU on),
blocks of 16 experts, pieces of 64 elements of d_model dealt to sixteen, eight or four wavefronts with a ring of two to four
pieces each, and top-k over up to 64 lanes.  Inputs are small integers with repeated gate rows, as in test_gpu_ties:
every logit is exact in fp32 in any order, so the routing and the observed workload must equal the oracle's."""
import numpy as np
import pytest
import torch

import paper_2503_06823_amd as P
import test_gpu_ties as ties
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

# (T, d_model, E, k, R, distinct gate rows)
CASES = [
    (1, 8, 1, 1, 1, 1), (1, 56, 16, 16, 16, 5), (15, 64, 17, 2, 9, 4), (16, 72, 16, 3, 9, 4), (17, 512, 15, 1, 6, 3),
    (31, 520, 33, 5, 20, 7), (33, 1032, 32, 32, 32, 9), (47, 1096, 49, 7, 30, 9), (64, 2048, 8, 2, 7, 3), (48, 2048, 9, 2, 7, 3),
    (18, 264, 64, 64, 64, 20), (4096, 136, 20, 2, 9, 4), (4097, 136, 10, 2, 7, 3), (4111, 328, 31, 3, 20, 8),
    (4129, 584, 48, 4, 31, 9), (8195, 264, 64, 6, 40, 12),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "T%d_d%d_E%d_k%d" % c[:4])
def test_gate_at_its_cuts(gpu_device, case):
    T, d, E, k, R, n_rows = case
    ties.test_equal_logits_go_to_the_lower_expert_index(gpu_device, (f"cuts_{case}", "bf16", T, d, E, k, R, n_rows, T % 2 == 1 and E > 1))


def test_infinite_and_nan_logits_leave_defined_choices(gpu_device):
    """A bias of -inf on all residents but two: the third choice is the lowest of the others, with weight 0.  A NaN comes after
    all numbers."""
    T, d, E, k, R = 21, 72, 20, 3, 12
    x, wg, _, soe = ties.tie_inputs("bf16", T, d, E, R, 9, False, seed=5)
    residents = np.flatnonzero(soe >= 0)
    a, b = residents[4], residents[9]
    te = torch.full((T, k), -7, dtype=torch.int32, device="cuda")
    tw = torch.full((T, k), -7.0, device="cuda")
    desc = P.make_desc(T, d, 64, E, k, R, "bf16", "swiglu")
    for low in (-np.inf, np.nan):
        bias = np.full(E, low, dtype=np.float32)
        bias[[a, b]] = 0.0
        P.emoe_route(desc, to_dev(x, "bf16"), to_dev(wg, "bf16"), torch.from_numpy(bias).cuda(), torch.from_numpy(soe).cuda(), te, tw)
        torch.cuda.synchronize()
        got, w = te.cpu().numpy(), tw.cpu().numpy()
        assert {frozenset(r) for r in got[:, :2].tolist()} == {frozenset((a, b))}
        assert (got[:, 2] == residents[0]).all()
        if np.isinf(low):
            assert (w[:, 2] == 0.0).all() and np.abs(w.sum(1) - 1.0).max() < 1e-6
