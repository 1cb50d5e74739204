"""The first product stores the hidden activations past the caches or plainly, by what passed through the GPU's memory since the
layer's last pass: same bits either way, in both entry points, at the tiles that do both and on either side of the rule."""
import pytest
import torch

from paper_2308_15030_amd import binding as b
from test_hidden_layout_gpu import layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,d,f,T,kernel,other", [
    # 101 MB of slots beside 201 MB of others: tiles of 32 and 64 rows
    (32, 512, 1536, 300, "grouped_gemm_bf16<1, 1", (16, 1024, 3072)), (32, 512, 1536, 1000, "grouped_gemm_bf16<1, 2", (16, 1024, 3072)),
    # 25 MB beside 134 MB: 256 x 256 tiles, several to a workgroup, ragged ends
    (16, 256, 1536, 8001, "ring_gemm_bf16_kept", (16, 1024, 2048)), (5, 320, 2048, 6000, "ring_gemm_bf16_kept", (16, 1024, 2048))])
def test_same_bits(K, d, f, T, kernel, other):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(K + d + f + T)
    o = layer(16, *other, 1, g)
    y = torch.zeros(1, other[1], dtype=torch.int16, device="cuda:0")
    L = layer(K, K, d, f, T, g)
    assert b.smoe_describe_ffn(L.handle, T).startswith(kernel)
    x = torch.randn(T, d, device="cuda:0", generator=g).to(torch.bfloat16).view(torch.int16)
    L.forward_fused(x, T, accumulate=0, residual=x)          # nothing but its own slots from here on
    want = L.forward_fused(x, T, accumulate=0, residual=x).clone()
    assert not torch.isnan(want.view(torch.bfloat16).float()).any()
    for call in (L.forward_fused, L.forward):
        o.forward_fused(y, 1, accumulate=0)
        assert b.smoe_describe_ffn(L.handle, T).startswith(kernel.replace("_kept", "<4, true>"))
        L.out.fill_(0)
        assert torch.equal(call(x, T, accumulate=0, residual=x), want)
    L.close()
    o.close()
