"""The layouts of the hidden activations between the two launches of a small batch (token by token, or unit by unit):
by the number of slots, by the width of d_ff, by whether the weights come from memory or from the cache, and behind a
router launch of its own.  Every output bit for bit against the five separate calls (which test_parity_gpu.py holds
against the oracle)."""
import pytest
import torch

from paper_2308_15030_amd import binding as b

pytestmark = pytest.mark.gpu

NAMES = ("orig_expert", "orig_gate", "slot", "gate", "xnorm", "count", "gsum", "score", "perm", "inv_perm", "offsets", "out")


def layer(E, K, d, f, T, g, spare=0):
    L = b.Layer(E, K, d, f, T, b.SMOE_BF16, router_w=torch.randn(E, d, device="cuda:0", generator=g) * d ** -0.5, device="cuda:0",
                spare_slots=spare)
    for k in range(K):
        L.set_resident(k, k, *(torch.randn(s, device="cuda:0", generator=g).mul_(0.05).to(torch.bfloat16) for s in ((d, f), (f, d))))
    return L


def check(L, x, T, want):
    for n in NAMES:
        getattr(L, n).fill_(0)
    L.forward_fused(x, T, accumulate=0, residual=x)
    for n in NAMES:
        assert torch.equal(getattr(L, n), want[n]), n


@pytest.mark.parametrize("E,K,d,f", [(8, 3, 96, 2080), (8, 4, 96, 2080), (16, 8, 96, 2080), (16, 8, 96, 2048), (16, 7, 64, 4128)])
@pytest.mark.parametrize("T,spare", [(17, 0), (32, 1), (33, 0), (64, 0), (65, 1), (128, 0)])
def test_from_cache_and_from_memory(E, K, d, f, T, spare):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(E + K + d + f + T)
    # a pass of this one is 201 MB of slot traffic: what L reads next does not come from the cache
    other = layer(16, 16, 1024, 3072, 1, g)
    y = torch.zeros(1, 1024, dtype=torch.int16, device="cuda:0")
    L = layer(E, K, d, f, T, g, spare)
    x = torch.randn(T, d, device="cuda:0", generator=g).to(torch.bfloat16).view(torch.int16)
    L.forward(x, T, accumulate=0, residual=x)
    want = {n: getattr(L, n).clone() for n in NAMES}
    assert not torch.isnan(want["out"].view(torch.bfloat16).float()).any()
    for stream in (False, True, False):
        if stream:
            other.forward_fused(y, 1, accumulate=0)
        assert ("_stream" in b.smoe_describe_ffn(L.handle, T)) == stream
        check(L, x, T, want)
    L.close()
    other.close()


@pytest.mark.parametrize("d,f,T", [(256, 3072, 17), (256, 3072, 32), (256, 3072, 33), (512, 3072, 64), (512, 3072, 65), (512, 2048, 33)])
def test_router_first(d, f, T):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(d + f + T)
    L = layer(64, 64, d, f, T, g)
    x = torch.randn(T, d, device="cuda:0", generator=g).to(torch.bfloat16).view(torch.int16)
    assert b.smoe_describe_ffn(L.handle, T).startswith("dense_first_kernel<")
    L.forward(x, T, accumulate=0, residual=x)
    want = {n: getattr(L, n).clone() for n in NAMES}
    assert not torch.isnan(want["out"].view(torch.bfloat16).float()).any()
    check(L, x, T, want)
    L.close()
