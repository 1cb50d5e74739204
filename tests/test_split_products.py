"""The second product with its reduction split over the waves of a workgroup (split_gemm_bf16): the rule that chooses it, and
the kernel where it can go wrong -- narrow last tiles, reductions too short for four parts or with parts of unequal length, empty
slots, more slots than a wave has lanes, several tiles per workgroup (small shapes), and every tile shape of 1 to 4 blocks either
way in long reductions, whose loops go round (`executed` below repeats the kernel's choice and says which run).

Forced through SMOE_FFN_VARIANT (11; read at smoe_create).  Reference and tolerance as in test_ring_gpu.py."""
import os

import numpy as np
import pytest
import torch

from paper_2308_15030_amd import binding as b
from test_streaming_tiles_gpu import MANY
from test_tile_choice import kernels


@pytest.mark.parametrize("K,d,f,T,kernel", [
    # small tiles, and larger ones while its own leave a fifth of the chip free
    (4, 768, 3072, 520, "split"), (16, 768, 3072, 777, "split"), (4, 768, 3072, 3750, "split"), (16, 768, 3072, 3100, "split"), (4, 768, 3072, 4096, "tiled"),
    (16, 768, 3072, 4096, "tiled"), (8, 768, 2048, 4096, "tiled"), (4, 768, 3072, 6000, "tiled"),
    # slots of less than a tile's rows
    (32, 1024, 4096, 800, "split"), (32, 768, 3072, 2000, "split"),
    # no multiple of 128; too short for the ring kernel
    (11, 416, 1696, 1213, "split"), (10, 992, 3296, 3100, "split"), (10, 992, 3296, 4000, "ring<2"), (10, 992, 3296, 6000, "ring<2"),
    (4, 64, 160, 1000, "split"), (4, 64, 160, 1000000, "tiled"),
    # large tiles for the chip many times over, whatever the rows of a slot
    (16, 768, 3072, 12000, "ring<4"), (128, 1024, 4096, 6000, "ring<4"), (128, 1024, 4096, 16000, "ring<4"), (16, 608, 2400, 12000, "ring<4"),
    # what streams stays so, but for wide rows
    (4, 768, 3072, 200, "streaming"), (16, 768, 3072, 60, "streaming"), (128, 9216, 256, 700, "streaming"), (128, 9216, 256, 760, "ring<4")])
def test_choice(K, d, f, T, kernel):
    name = {"split": "split_gemm_bf16", "tiled": "grouped_gemm_bf16<", "streaming": "small_gemm_bf16<4, 4"}.get(kernel, kernel.replace("ring", "ring_gemm_bf16"))
    assert kernels(K, d, f, T)[1].startswith(name)


def executed(lens, N, R, per_die=32):
    """Tile shapes (feature, token blocks) that the kernel runs on these segments, and the one that it picks."""
    nfb, per = N // 32, -(-(R // 16) // 4)
    items = (sum(lens) // 32 + len(lens)) * nfb
    nwg = max(min(-(-items // 8), per_die), 1)
    blocks = [-(-n // 32) for n in lens]
    def price(w, h):
        tiles = sum(-(-b // h) for b in blocks) * -(-nfb // w)
        return -(-(-(-tiles // 8)) // nwg) * (per * (15 * (w + h) + 4 * w * h) + 157 * w * h)
    W, H = min(((w, h) for w in range(1, 5) for h in range(1, 5)), key=lambda s: price(*s))
    cut = lambda n, most: {n // -(-n // most) + (i < n % -(-n // most)) for i in range(-(-n // most))}
    return (W, H), {(w, h) for b in blocks if b for w in cut(nfb, W) for h in cut(b, H)}


# (segments, d_model, d_ff): each is the pick of one shape, evenly or unevenly cut, with parts of 24 steps and more
LONG = [([1], 768, 3072), ([97, 128, 129, 300], 384, 3072), ([97, 128, 129, 300], 768, 3072), ([120] * 48, 160, 1696), ([412, 88], 992, 1632),
        ([1500, 40, 700], 384, 3072), ([1500, 40, 700], 512, 2048), ([1500, 40, 700], 768, 3072), ([97, 128, 129, 300], 992, 3296),
        ([1300, 700, 33, 1950], 384, 3072), ([190] * 16, 768, 3072), ([1000] * 4, 768, 3072), ([858, 142], 992, 1632), ([1300, 700, 33, 1950], 992, 3296),
        ([190] * 16, 992, 3296), ([900, 100, 640, 31, 0, 333, 517, 64, 1200, 215], 768, 3072)]
SHAPES = [(w, h) for w in range(1, 5) for h in range(1, 5)]


def test_every_shape_is_run():
    assert [executed(*c)[0] for c in LONG] == SHAPES
    assert {s for c in LONG for s in executed(*c)[1]} == set(SHAPES)
    assert any(len(executed(*c)[1]) > 2 for c in LONG)


@pytest.mark.gpu
@pytest.mark.parametrize("lens,d,f", LONG, ids=[f"{w}x{h}" for w, h in SHAPES])
def test_long_reductions(lens, d, f):
    check(lens, d, f)


@pytest.mark.gpu
@pytest.mark.parametrize("lens", [[1], [0, 31, 0, 33, 64, 0], [97, 128, 129, 300], [1500, 40, 700], MANY, [5] * 200],
                         ids=["one", "empty", "edges", "large", "many", "thin"])
# (d_model, d_ff): 1 to 5 and 25 feature blocks; reductions of 2, 6, 10, 18 and 106 steps of 16
@pytest.mark.parametrize("d,f", [(32, 32), (64, 96), (96, 160), (160, 288), (128, 1696), (800, 288)])
def test_split_products(d, f, lens):
    check(lens, d, f)


def check(lens, d, f):
    K, T, dev = len(lens), sum(lens), "cuda:0"
    g = torch.Generator(device=dev)
    g.manual_seed(d + f + T)
    E = max(8, K)
    os.environ["SMOE_FFN_VARIANT"] = "1,11"
    try:
        L = b.Layer(E, K, d, f, T, b.SMOE_BF16, router_w=torch.randn(E, d, device=dev, generator=g) * 0.1, device=dev, spare_slots=K % 2)
    finally:
        del os.environ["SMOE_FFN_VARIANT"]
    if T > 128:
        assert b.smoe_describe_ffn(L.handle, T, False).endswith(" | split_gemm_bf16")
    w1 = (torch.randn(K, d, f, device=dev, generator=g) * d ** -0.5).to(torch.bfloat16)
    w2 = (torch.randn(K, f, d, device=dev, generator=g) * f ** -0.5).to(torch.bfloat16)
    for k in range(K):
        L.set_resident(k, k, w1[k], w2[k])
    x = torch.randn(T, d, device=dev, generator=g).to(torch.bfloat16)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    L.x_perm.copy_(x.view(torch.int16))
    L.offsets.copy_(torch.from_numpy(off))
    L.y_perm.fill_(0x7fc0)                                   # a NaN where nothing is written
    L.expert_ffn(T)
    got = L.y_perm.view(torch.bfloat16).float()
    for k in range(K):
        a, e = int(off[k]), int(off[k + 1])
        if a == e:
            continue
        ref = (x[a:e].float() @ w1[k].float()).relu().to(torch.bfloat16).float() @ w2[k].float()
        assert (got[a:e] - ref).abs().max() <= 2e-2 * ref.abs().max(), (k, lens[k])
    # the single-call layer (rows scattered with gate and residual) gives the bits of the separate calls, with and without residual
    x = x.view(torch.int16)
    for res in (x, None):
        out = L.forward(x, T, accumulate=0, residual=res).clone()
        L.out.fill_(0)
        assert torch.equal(L.forward_fused(x, T, accumulate=0, residual=res), out)
    L.close()
