"""The second product with its reduction split over the waves of a workgroup (split_gemm_bf16): the rule that chooses it, and
the kernel where it can go wrong -- every tile shape of 1 to 4 blocks either way, narrow last tiles, reductions too short for
four parts or with parts of unequal length, empty slots, more slots than a wave has lanes, several tiles per workgroup.

Forced through SMOE_FFN_VARIANT (11; read at smoe_create).  Reference and tolerance as in test_ring_gpu.py."""
import os

import numpy as np
import pytest
import torch

from paper_2308_15030_amd import binding as b
from test_streaming_tiles_gpu import MANY
from test_tile_choice import kernels


@pytest.mark.parametrize("K,d,f,T,split", [
    # instead of tiles of 32 and 64 rows; instead of 128 x 128 tiles while its own leave a fifth of the chip free
    (4, 768, 3072, 520, True), (16, 768, 3072, 777, True), (4, 768, 3072, 4000, True), (16, 768, 3072, 3100, True), (4, 768, 3072, 4096, False),
    (16, 768, 3072, 4096, False), (8, 768, 2048, 4096, False), (4, 768, 3072, 6000, False),
    # slots of less than a tile's rows
    (32, 1024, 4096, 800, True), (32, 768, 3072, 2000, True),
    # no multiple of 128
    (11, 416, 1696, 1213, True), (10, 992, 3296, 4000, True), (10, 992, 3296, 6000, False),
    # what streams stays so
    (4, 768, 3072, 200, False), (16, 768, 3072, 60, False)])
def test_choice(K, d, f, T, split):
    assert (kernels(K, d, f, T)[1] == "split_gemm_bf16") == split


@pytest.mark.gpu
@pytest.mark.parametrize("lens", [[1], [0, 31, 0, 33, 64, 0], [97, 128, 129, 300], [1500, 40, 700], MANY, [5] * 200],
                         ids=["one", "empty", "edges", "large", "many", "thin"])
# (d_model, d_ff): 1 to 5 and 25 feature blocks; reductions of 2, 6, 10, 18 and 106 steps of 16
@pytest.mark.parametrize("d,f", [(32, 32), (64, 96), (96, 160), (160, 288), (128, 1696), (800, 288)])
def test_split_products(d, f, lens):
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
