"""The streaming products (small_gemm_bf16) with slots of more than 32 tokens: the first 32 rows of a slot and its
further row tiles are different workgroups, the latter found by counting through the slots.

Forced through SMOE_FFN_VARIANT (5 = whole reduction, 6 = split four ways; read at smoe_create).  Segments: everything
in one slot, with and without a remainder (the bound on the further tiles is then reached); slots of 0 to 10 row tiles on
both sides of slots 64 and 128, where the count goes on from one chunk of 64 slots to the next.
Reference and tolerance as in test_ring_gpu.py."""
import os

import numpy as np
import pytest
import torch

from paper_2308_15030_amd import binding as b

pytestmark = pytest.mark.gpu

MANY = [0] * 130
for _k, _n in {0: 1, 5: 33, 62: 64, 63: 300, 64: 65, 65: 31, 100: 32, 127: 97, 128: 40, 129: 129}.items():
    MANY[_k] = _n


@pytest.mark.parametrize("variant", ["5,5", "6,6"])
@pytest.mark.parametrize("d,f", [(96, 160), (256, 288)])
@pytest.mark.parametrize("lens", [[160], [161], [0, 0, 191], [1, 32, 33, 64, 65, 5], MANY], ids=["whole", "remainder", "last", "few", "many"])
def test_row_tiles(variant, d, f, lens, kernel="small_gemm_bf16"):
    K, T, dev = len(lens), sum(lens), "cuda:0"
    g = torch.Generator(device=dev)
    g.manual_seed(d + f + T)
    E = max(8, K)
    os.environ["SMOE_FFN_VARIANT"] = variant
    try:
        L = b.Layer(E, K, d, f, T, b.SMOE_BF16, router_w=torch.randn(E, d, device=dev, generator=g) * 0.1, device=dev, spare_slots=K % 2)
    finally:
        del os.environ["SMOE_FFN_VARIANT"]
    assert b.smoe_describe_ffn(L.handle, T, False).count(kernel) == 2
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
    # the single-call layer, which gathers and scatters the rows in the products
    x = x.view(torch.int16)
    out = L.forward(x, T, accumulate=0, residual=x).clone()
    L.out.fill_(0)
    assert torch.equal(L.forward_fused(x, T, accumulate=0, residual=x), out)
    L.close()
