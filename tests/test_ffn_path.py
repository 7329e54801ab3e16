"""Which kernels the bf16 FFN of a layer takes, at layers where the times of the two tile sizes were measured to be apart
and on both sides of the rows per slot at which the choice may change; which layers leave the sort to their first
product, where that was measured to be faster, or slower; and which products of up to 16 tokens the streaming kernels take."""
import ctypes

import pytest

import paper_2503_06823_amd as P
from gpu_util import F32, FEW, MID, STREAM, TILED, ffn_kernels, ffn_path


@pytest.mark.parametrize("rows,small,large", [(1, STREAM, STREAM), (22, STREAM, STREAM), (23, MID, MID), (100, MID, MID),
                                              (101, MID, TILED), (169, MID, TILED), (170, MID, TILED), (300, MID, TILED),
                                              (301, TILED, TILED), (4000, TILED, TILED)])
def test_rows_per_slot(rows, small, large):
    for S in (1, 4, 8):
        assert ffn_path(P.make_desc(rows * S, 256, 512, S, 1, S, "bf16", "swiglu")) == small
        assert ffn_path(P.make_desc(rows * S, 4096, 14336, S, 1, S, "bf16", "swiglu")) == large
    assert ffn_path(P.make_desc(rows * 4, 256, 512, 8, 2, 8, "bf16", "relu")) == small  # A = T * k


# d_model, d_ff, slots, rows per slot, activation: where tiles of 128 (MID) or of 256 rows were the faster ones, by 10 % or more
FASTER = [
    # 100 to 169 rows per slot
    (2048, 1408, 4, 128, "swiglu", MID), (768, 3072, 4, 160, "swiglu", MID), (1536, 1536, 8, 160, "swiglu", MID),
    (1040, 1048, 8, 160, "swiglu", MID), (1032, 2808, 4, 128, "relu", MID), (1024, 2816, 8, 160, "relu", MID),
    (2048, 1408, 8, 160, "relu", MID), (512, 1408, 32, 128, "relu", MID), (4104, 2056, 1, 160, "swiglu", MID),
    (1536, 1536, 12, 128, "relu", MID), (6144, 2048, 2, 128, "relu", MID), (2048, 8192, 1, 160, "swiglu", MID),
    (520, 4104, 12, 128, "relu", TILED), (520, 4104, 8, 160, "relu", TILED), (520, 4104, 8, 160, "swiglu", TILED),
    (4104, 2056, 2, 128, "swiglu", TILED), (2056, 4104, 2, 140, "swiglu", TILED), (2056, 4104, 2, 166, "swiglu", TILED),
    (520, 6152, 8, 140, "relu", TILED), (6152, 520, 8, 140, "relu", TILED), (512, 4096, 8, 118, "swiglu", TILED),
    (640, 5120, 4, 140, "swiglu", TILED), (640, 5120, 8, 140, "relu", TILED), (520, 6152, 4, 140, "swiglu", TILED),
    (4096, 4096, 2, 128, "relu", TILED), (4104, 2056, 4, 128, "relu", TILED),
    # 170 to 300
    (2048, 1408, 8, 200, "swiglu", MID), (2048, 1408, 8, 256, "swiglu", MID), (768, 3072, 16, 200, "relu", MID),
    (2048, 8192, 2, 200, "relu", MID), (1536, 1536, 16, 256, "relu", MID), (6144, 2048, 2, 200, "swiglu", MID),
    (1024, 2816, 8, 200, "swiglu", MID), (512, 1408, 32, 200, "swiglu", MID), (1536, 4096, 8, 200, "relu", MID),
    # weights above the limits
    (4096, 14336, 8, 256, "swiglu", TILED), (4096, 14336, 4, 128, "swiglu", TILED), (4104, 4096, 4, 128, "swiglu", TILED),
]


@pytest.mark.parametrize("d,f,S,rows,act,path", FASTER)
def test_faster_tiles_are_chosen(d, f, S, rows, act, path):
    assert ffn_path(P.make_desc(rows * S, d, f, S, 1, S, "bf16", act)) == path


def test_the_kernels_of_a_layer():
    for S, k in ((1, 1), (8, 2), (64, 64)):
        assert ffn_kernels(P.make_desc(1, 256, 512, S, k, S, "f32", "swiglu")) == F32
        for T in (1, 16):
            assert ffn_kernels(P.make_desc(T, 4096, 14336, S, k, S, "bf16", "swiglu")) == FEW
        for T in (17, 22, 200, 5000):
            desc = P.make_desc(T, 1024, 2048, S, k, S, "bf16", "relu")
            assert ffn_kernels(desc) == ffn_path(desc)
            assert ffn_kernels(P.make_desc(T, 1024, 2048, S, k, S, "f32", "relu")) == F32


class DeviceShape(ctypes.Structure):
    _fields_ = [("cus", ctypes.c_int), ("xcds", ctypes.c_int), ("groups", ctypes.c_int)]


def sorts(*args):
    fn = getattr(P.lib(), "_ZN4emoe19first_product_sortsERK15emoe_layer_descRKNS_11DeviceShapeE")
    fn.restype = ctypes.c_bool
    return fn(ctypes.byref(P.make_desc(*args)), ctypes.byref(DeviceShape(256, 8, 256)))


# T, d_model, d_ff, E, k, S, dtype, activation
SLOWER = [
    # streaming, one pass, short walks
    (29, 64, 1344, 42, 3, 41, "bf16", "swiglu"), (30, 384, 1664, 37, 1, 35, "bf16", "swiglu"), (29, 128, 2560, 30, 2, 25, "bf16", "swiglu"),
    (34, 192, 1920, 58, 7, 33, "bf16", "swiglu"), (25, 128, 7040, 23, 1, 18, "bf16", "relu"), (94, 72, 6784, 53, 1, 16, "bf16", "relu"),
    (120, 768, 3072, 64, 8, 64, "bf16", "swiglu"), (256, 4096, 14336, 8, 2, 8, "bf16", "swiglu"),
    (342, 1024, 2048, 8, 3, 8, "bf16", "swiglu"), (1025, 64, 64, 1, 1, 1, "f32", "relu"),  # more than 1024 assignments
    (1024, 4096, 4096, 2, 1, 2, "bf16", "swiglu"),                                          # the 256-row tiles do not sort
]
FASTER_SORTING = [
    (64, 128, 256, 8, 2, 4, "f32", "swiglu"), (1, 4096, 14336, 8, 2, 6, "bf16", "swiglu"), (300, 1024, 1024, 8, 3, 8, "bf16", "swiglu"),
    (95, 544, 472, 57, 4, 55, "bf16", "swiglu"), (100, 864, 1176, 24, 3, 21, "bf16", "swiglu"), (90, 400, 864, 35, 4, 29, "bf16", "swiglu"),
]


@pytest.mark.parametrize("layer,where", [(l, False) for l in SLOWER] + [(l, True) for l in FASTER_SORTING], ids=str)
def test_the_sort_goes_where_it_is_faster(layer, where):
    assert sorts(*layer) == where


# SwiGLU, rows, slots, outputs, inputs, streaming.  Where weight rows are whole lines, walks short, units few or the rows per slot
# few, the few-token kernel was the faster one.
PRODUCTS = [
    (True, 28, 2, 15816, 3208, True), (True, 39, 3, 10744, 4816, True), (True, 32, 3, 14544, 4568, True), (True, 15, 1, 5200, 5608, True),
    (True, 28, 2, 5376, 3208, False), (True, 28, 2, 15816, 3200, False), (True, 6, 2, 15816, 3208, False), (True, 28, 2, 2048, 3208, False),
    (False, 28, 2, 3208, 15816, True), (False, 7, 7, 1752, 16120, False), (False, 16, 8, 552, 13304, True), (False, 10, 10, 552, 13304, False),
    (False, 28, 2, 3208, 15808, False), (False, 28, 2, 2040, 15816, False), (False, 28, 2, 3208, 2040, False), (False, 7, 1, 16384, 4104, True),
    (False, 16, 8, 5216, 11208, False), (False, 36, 6, 5216, 11208, True), (False, 6, 6, 5216, 11208, False), (False, 48, 6, 8000, 11208, False),
]


@pytest.mark.parametrize("product", PRODUCTS, ids=str)
def test_few_token_products_that_stream(product):
    fn = getattr(P.lib(), "_ZN4emoe19few_product_streamsEbxiiii")
    fn.restype, fn.argtypes = ctypes.c_bool, [ctypes.c_bool, ctypes.c_longlong] + [ctypes.c_int] * 4
    assert fn(*product[:5], 256) == product[5]
