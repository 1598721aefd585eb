"""Which tile and how many splits of the reduction the large-M GEMM takes (a
host rule on the shape, no GPU): the tiles that the GPU tests of whole models
mean to run, and those of the 7B, 13B and 70B shapes.  Between them every tile
and every kind of product occurs."""

import ctypes

import pytest

from paper_2309_08168_amd import binding

STORE, RESID, SWIGLU, QKV = 0, 1, 2, 3


def tile(M, N, K, epi):
    lib = binding.load()
    bn, bm, splits = (ctypes.c_int32() for _ in range(3))
    assert lib.sdk_prefill_tile(M, N, K, epi, ctypes.byref(bn), ctypes.byref(bm), ctypes.byref(splits)) >= 0
    return bn.value, bm.value, splits.value


def products(d, hd, nq, F, vocab):
    """(kind, N, K) of a model's products."""
    return {"qkv": (QKV, nq, d), "o": (RESID, d, hd), "gate_up": (SWIGLU, 2 * F, d), "down": (RESID, d, F),
            "head": (STORE, vocab, d)}


SHAPES = {
    "7b": (4096, 4096, 12288, 11008, 32000),
    "13b": (5120, 5120, 15360, 13824, 32000),
    "70b": (8192, 8192, 10240, 28672, 32000),
    # models of test_gpu_prefill.py and test_gpu_prefill_terms.py
    "ffn_wide_bf16": (256, 256, 768, 7200, 512),
    "d2560_bf16": (2560, 2560, 7680, 2048, 512),
    "split_wide_bf16": (5120, 1024, 3072, 4096, 512),
    "all_wide_bf16": (256, 12288, 16384, 7200, 16381),
    "terms_thin": (256, 256, 512, 1344, 777),
    "terms_ragged": (136, 96, 160, 200, 777),
    "terms_long_k": (512, 256, 512, 2048, 400),
}


@pytest.mark.parametrize("name,rows,product,want", [
    ("13b", 1023, "qkv", (256, 256, 1)),
    ("13b", 1023, "gate_up", (224, 256, 1)),
    ("13b", 1023, "o", (256, 256, 3)),
    ("13b", 1023, "down", (256, 256, 3)),
    ("7b", 511, "qkv", (256, 128, 1)),
    ("7b", 511, "gate_up", (224, 256, 1)),
    ("7b", 511, "o", (256, 128, 4)),
    ("13b", 129, "qkv", (128, 128, 1)),
    ("13b", 129, "head", (256, 128, 1)),
    ("13b", 100, "qkv", (128, 64, 1)),
    ("13b", 100, "down", (128, 128, 6)),
    ("ffn_wide_bf16", 600, "gate_up", (224, 256, 1)),
    ("ffn_wide_bf16", 1000, "gate_up", (256, 256, 1)),
    ("ffn_wide_bf16", 1024, "gate_up", (256, 256, 1)),
    ("d2560_bf16", 1000, "o", (256, 128, 3)),
    ("d2560_bf16", 1000, "down", (256, 128, 3)),
    ("split_wide_bf16", 1000, "down", (256, 256, 3)),
    ("all_wide_bf16", 1000, "qkv", (256, 256, 1)),
    ("all_wide_bf16", 1000, "head", (256, 256, 1)),
    ("terms_thin", 513, "gate_up", (128, 64, 1)),
    ("terms_ragged", 513, "down", (128, 64, 1)),
])
def test_tile_of_a_shape(name, rows, product, want):
    epi, N, K = products(*SHAPES[name])[product]
    assert tile(rows, N, K, epi) == want


@pytest.mark.parametrize("rows", [1, 17, 65, 300, 512, 513, 1000, 1024])
def test_splits_stay_within_the_scratch(rows):
    """At most 8 planes of partial sums, 4096 rows of them in all, at least 8 stages of 32 each; one for the others."""
    for shape in SHAPES.values():
        for epi, N, K in products(*shape).values():
            splits = tile(rows, N, K, epi)[2]
            assert 1 <= splits <= (8 if epi == RESID else 1)
            assert splits * rows <= 4096
            assert splits == 1 or -(-K // 32) >= 8 * splits


@pytest.mark.parametrize("M,N,K", [(0, 64, 64), (1025, 64, 64), (17, 0, 64), (17, 64, 0)])
def test_shapes_out_of_range_are_refused(M, N, K):
    out = [ctypes.byref(ctypes.c_int32()) for _ in range(3)]
    assert binding.load().sdk_prefill_tile(M, N, K, RESID, *out) == -1
