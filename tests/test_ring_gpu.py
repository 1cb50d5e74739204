"""The ring kernel of the prefill products (ring_gemm_bf16) where it can go wrong.

Forced through SMOE_FFN_VARIANT (read once, at smoe_create; 9 = tiles of at most
128 x 128, 10 = at most 256 x 256): the shortest reduction it takes (8 slices),
odd slice counts, feature counts that leave the last tile narrow, segments of
1 to several tiles with empty slots between them, and enough items that a
workgroup walks several (the loads run on from one tile into the next).
Reference: the two products in fp32 with the hidden activations rounded to
bf16, as the library rounds them; the tolerance covers one more rounding of a
value near a rounding boundary (2**-8 of the largest) and the output's own.
"""
import os

import numpy as np
import pytest
import torch

from paper_2308_15030_amd import binding as b
from test_streaming_tiles_gpu import MANY, test_row_tiles as check

pytestmark = pytest.mark.gpu

SEGMENTS = [1, 0, 33, 256, 257, 31, 0, 700]


@pytest.mark.parametrize("variant", [9, 10])
# (d_model, d_ff, extra tokens of the last slot): reductions of 8 slices; of odd counts (13, 53); first product of
# several items per workgroup (32 feature tiles); second product likewise (8 feature tiles, 290 row blocks)
@pytest.mark.parametrize("d,f,extra", [(256, 256, 0), (416, 1696, 100), (256, 8192, 1800), (2048, 288, 8000)])
@pytest.mark.parametrize("spare", [0, 1])
def test_ring_products(variant, d, f, extra, spare):
    lens = list(SEGMENTS)
    lens[-1] += extra
    K, T, dev = len(lens), sum(lens), "cuda:0"
    g = torch.Generator(device=dev)
    g.manual_seed(7 * d + f)
    os.environ["SMOE_FFN_VARIANT"] = f"{variant},{variant}"
    try:
        L = b.Layer(16, K, d, f, T, b.SMOE_BF16, router_w=torch.randn(16, d, device=dev, generator=g) * 0.1, device=dev,
                    spare_slots=spare)
    finally:
        del os.environ["SMOE_FFN_VARIANT"]
    assert b.smoe_describe_ffn(L.handle, T, False).count("ring_gemm_bf16") == 2
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
        h = (x[a:e].float() @ w1[k].float()).relu().to(torch.bfloat16).float()
        ref = h @ w2[k].float()
        assert (got[a:e] - ref).abs().max() <= 2e-2 * ref.abs().max(), (k, lens[k])
    # the single-call layer (rows gathered and scattered in the products) gives the bits of the separate calls
    out = L.forward(x.view(torch.int16), T, accumulate=0, residual=x.view(torch.int16)).clone()
    L.out.fill_(0)
    assert torch.equal(L.forward_fused(x.view(torch.int16), T, accumulate=0, residual=x.view(torch.int16)), out)
    assert not torch.isnan(out.view(torch.bfloat16).float()).any()
    L.close()


# more slots than a wave has lanes: the counts of row tiles and the slot tables go on from one chunk of 64 slots to the next
@pytest.mark.parametrize("variant", ["9,9", "10,10"])
@pytest.mark.parametrize("d,f", [(256, 288), (288, 544)])
@pytest.mark.parametrize("lens", [MANY, [0] * 63 + [40, 700], [300] + [0] * 200 + [33], [5] * 256], ids=["many", "64th", "last", "all"])
def test_many_slots(variant, d, f, lens):
    check(variant, d, f, lens, "ring_gemm_bf16")
