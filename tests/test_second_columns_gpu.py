"""smoe_forward on small batches whose second product needs several blocks of 32 columns for a slot: all tokens on one
slot, slots with exactly 32, 33 and 64 of them, and both layouts of the hidden activations between the launches (by
token, from four slots of more than 2048 hidden features on; by unit otherwise).  Every output bit for bit against the
five separate calls (which test_parity_gpu.py holds against the oracle)."""
import numpy as np
import pytest
import torch

from paper_2308_15030_amd import binding as b

pytestmark = pytest.mark.gpu

NAMES = ("orig_expert", "orig_gate", "slot", "gate", "xnorm", "count", "gsum", "score", "perm", "inv_perm", "offsets", "out")


@pytest.mark.parametrize("d,f", [(96, 256), (64, 2080)])
@pytest.mark.parametrize("counts", [[33, 0, 0, 0], [64, 0, 0, 0], [128, 0, 0, 0], [1, 32, 33, 62], [0, 65, 0, 63], [31, 1, 0, 0], [32, 64], [127]])
@pytest.mark.parametrize("spare", [0, 1])
def test_columns(d, f, counts, spare):
    K, T, dev = len(counts), sum(counts), "cuda:0"
    g = torch.Generator(device=dev)
    g.manual_seed(d + f + T)
    L = b.Layer(8, K, d, f, T, b.SMOE_BF16, device=dev, spare_slots=spare)
    # a token's first K columns name its slot, and the router's rows of the resident experts read them
    L.router_w.zero_()
    L.router_w[:K, :K] = torch.eye(K, device=dev) * 8
    for k in range(K):
        L.set_resident(k, k, *(torch.randn(s, device=dev, generator=g).mul_(0.1).to(torch.bfloat16) for s in ((d, f), (f, d))))
    want = torch.tensor(np.random.default_rng(T).permutation(np.repeat(np.arange(K), counts)), device=dev)
    x = torch.randn(T, d, device=dev, generator=g)
    x[:, :K] = torch.nn.functional.one_hot(want, K).float() * 4
    x = x.to(torch.bfloat16).view(torch.int16)
    assert b.smoe_describe_ffn(L.handle, T).split(" | ")[1].startswith("decode_second")
    L.forward_fused(x, T, accumulate=0, residual=x)
    got = {n: getattr(L, n).clone() for n in NAMES}
    assert torch.equal(got["slot"], want.int())
    for n in NAMES:
        getattr(L, n).fill_(0)
    L.forward(x, T, accumulate=0, residual=x)
    for n in NAMES:
        assert torch.equal(getattr(L, n), got[n]), n
    assert not torch.isnan(got["out"].view(torch.bfloat16).float()).any()
    L.close()
