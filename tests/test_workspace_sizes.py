"""The FFN workspace that a bf16 layer is told to bring, over row counts and weight sizes: callers keep these sizes, so a
change of the rules that choose the kernels must not ask for more."""
import pytest

import paper_2503_06823_amd as P

MIB = 1 << 20
NONE, SMALLER, LARGER = 0, 32 * MIB, 256 + 64 * MIB  # beside h: streamed; K pieces of 128-row tiles; of 256-row tiles and their plan

# d_model, d_ff, S, activation: the weights of all slots
LAYERS = {
    "1 MiB": (128, 256, 4, "swiglu"),
    "108 MiB": (768, 3072, 8, "swiglu"),
    "112 MiB": (2048, 7168, 2, "relu"),
    "132 MiB": (2048, 1408, 8, "swiglu"),
    "176 MiB": (2048, 1408, 16, "relu"),
    "198 MiB": (2048, 1408, 12, "swiglu"),
    "288 MiB": (768, 3072, 32, "relu"),
    "320 MiB": (4096, 4096, 5, "relu"),
    "321 MiB": (4096, 4104, 5, "relu"),
    "2688 MiB": (4096, 14336, 8, "swiglu"),
}
SMALL = {"1 MiB", "108 MiB", "112 MiB", "132 MiB", "176 MiB", "198 MiB", "288 MiB", "320 MiB"}


@pytest.mark.parametrize("layer", LAYERS)
@pytest.mark.parametrize("rows,beside_h_small,beside_h", [
    (1, NONE, NONE), (22, NONE, NONE), (23, SMALLER, SMALLER), (100, SMALLER, SMALLER), (101, LARGER, LARGER),
    (169, LARGER, LARGER), (170, SMALLER, LARGER), (200, SMALLER, LARGER), (256, SMALLER, LARGER), (300, SMALLER, LARGER),
    (301, LARGER, LARGER), (1000, LARGER, LARGER)])
def test_workspace_beside_h(layer, rows, beside_h_small, beside_h):
    d, f, S, act = LAYERS[layer]
    T = rows * S
    size = P.emoe_workspace_bytes(P.make_desc(T, d, f, S, 1, S, "bf16", act))[1]
    assert size - (T * f * 2 + 255) // 256 * 256 == (beside_h_small if layer in SMALL else beside_h)
