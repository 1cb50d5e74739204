"""fp32 expert FFN with two workgroups of 4 waves per compute unit (each wave takes two of the eight parts of the
reduction): segments of one row to several row tiles, empty slots, every width of the feature range, reductions with
empty and odd parts.  Against the products in float64; the tolerance is the parity tests' 1e-4 of the tensor's scale."""
import numpy as np
import pytest
import torch

from paper_2308_15030_amd import binding as b

pytestmark = pytest.mark.gpu


#                         d    f     segments (at least 48 tokens per slot on average, more than 256 items of a product)
@pytest.mark.parametrize("d,f,lens", [(64, 4096, [1, 0, 255, 33, 17, 250]), (132, 2052, [700, 0, 16]), (20, 8192, [97, 1]),
                                      (4096, 68, [900, 3, 31, 1100]), (300, 1200, [128, 128])])
def test_pairs(d, f, lens):
    K, T, dev = len(lens), sum(lens), "cuda:0"
    g = torch.Generator(device=dev)
    g.manual_seed(d + f)
    L = b.Layer(8, K, d, f, T, b.SMOE_F32, router_w=torch.randn(8, d, device=dev, generator=g), device=dev)
    w1 = torch.randn(K, d, f, device=dev, generator=g) * d ** -0.5
    w2 = torch.randn(K, f, d, device=dev, generator=g) * f ** -0.5
    for k in range(K):
        L.set_resident(k, k, w1[k], w2[k])
    x = torch.randn(T, d, device=dev, generator=g)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    L.x_perm.copy_(x)
    L.offsets.copy_(torch.from_numpy(off))
    L.y_perm.fill_(float("nan"))
    L.expert_ffn(T)
    got = L.y_perm.double().cpu()
    for k in range(K):
        a, e = int(off[k]), int(off[k + 1])
        if a < e:
            ref = (x[a:e].double().cpu() @ w1[k].double().cpu()).relu() @ w2[k].double().cpu()
            assert (got[a:e] - ref).abs().max() <= 1e-4 * ref.abs().max(), (k, lens[k])
    L.close()


@pytest.mark.parametrize("d,f", [(64, 4096), (4096, 68), (132, 2052)])
def test_a_rows_bits_do_not_depend_on_the_batch(d, f):
    """The parts are added in the same order by 4 and by 8 waves: rows of a large batch (4 waves in one product or in
    both) against the same rows in a batch of a few tokens (8 waves)."""
    lens, few, dev = [200, 0, 190, 210], 9, "cuda:0"
    K, T = len(lens), sum(lens)
    g = torch.Generator(device=dev)
    g.manual_seed(d * 3 + f)
    L = b.Layer(8, K, d, f, T, b.SMOE_F32, router_w=torch.randn(8, d, device=dev, generator=g), device=dev)
    for k in range(K):
        L.set_resident(k, k, torch.randn(d, f, device=dev, generator=g) * d ** -0.5, torch.randn(f, d, device=dev, generator=g) * f ** -0.5)
    x = torch.randn(T, d, device=dev, generator=g)

    def ffn(rows, lens):
        n = sum(lens)
        L.x_perm[:n].copy_(rows)
        L.offsets.copy_(torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)))
        L.y_perm.fill_(float("nan"))
        L.expert_ffn(n)
        return L.y_perm[:n].clone()

    whole = ffn(x, lens)
    start = np.concatenate([[0], np.cumsum(lens)])
    at = torch.tensor([int(start[k]) + 17 + i for k in range(K) if lens[k] for i in range(few)], device=dev)
    assert torch.equal(ffn(x[at], [few if n else 0 for n in lens]), whole[at])
    L.close()
