"""Which kernels the separate FFN call and a prefill batch take, at the lines of the rules in pick_variants.  (No GPU: the
choice is made from the sizes.)"""
import pytest

from paper_2308_15030_amd import binding as b


def kernels(K, d, f, T, fused=False):
    h = b.smoe_create(max(K, 2), K, d, f, T, b.SMOE_BF16)
    try:
        return b.smoe_describe_ffn(h, T, fused).split(" | ")
    finally:
        b.smoe_destroy(h)


@pytest.mark.parametrize("K,d,f,T,streams", [
    # few slots, whatever their weights and however many tokens a slot has
    (6, 512, 2048, 132, True), (4, 768, 3072, 200, True), (2, 768, 3072, 140, True), (1, 768, 3072, 400, True),
    # d_model = 768, 24 workgroups per row tile: up to 700 from 28 tokens per slot on, below 780, or 850 with
    # long reductions and 14 tokens per slot
    (14, 768, 3072, 480, True), (15, 768, 3072, 480, False), (16, 768, 3072, 448, False), (17, 768, 3072, 448, True),
    (20, 768, 3072, 480, True), (21, 768, 3072, 480, False), (18, 768, 2048, 448, True), (19, 768, 2048, 448, False), (26, 768, 3072, 223, True), (27, 768, 3072, 223, False),
    (32, 768, 3072, 236, False),
    # short reductions and many tokens
    (8, 256, 768, 140, True), (8, 256, 640, 140, False), (2, 512, 2048, 512, True), (2, 512, 2048, 513, False),
    # up to five tokens per slot always
    (100, 512, 2048, 590, True)])
def test_second_product_streams(K, d, f, T, streams):
    assert kernels(K, d, f, T)[1].startswith("small_gemm_bf16<4, 4") == streams


@pytest.mark.parametrize("K,d,f,T,streams", [
    # d_model no multiple of 64, fewer than six tokens per slot
    (24, 992, 3296, 100, True), (64, 992, 3296, 380, True), (65, 992, 3296, 380, False), (24, 864, 3456, 130, False),
    (32, 416, 1696, 150, False), (24, 992, 3296, 144, False)])
def test_first_product_streams(K, d, f, T, streams):
    assert kernels(K, d, f, T)[0].startswith("small_gemm_bf16<4, 1" if streams else "ring_gemm_bf16")
