"""The router at widths where some of its reduction slices have no step (d_model = 96, 416 and 1056 with
eight slices, 32 and 96 with four): nothing behind the packed router weights may reach a product.  The
workspace and 4 KiB behind it are all NaN (0xFF bytes) before anything is put into it, and the layer's
expert norms are given, so that no call of this handle overwrites what follows the weights.  Against the oracle:
choices exactly outside near-ties, gates and norms at 1e-5, outputs at the bf16 tolerance of the parity tests."""
import numpy as np
import pytest
import torch

import oracle
from paper_2308_15030_amd import binding as b
from paper_2308_15030_amd import workloads as wl
from harness import max_abs_rel, to_dev, to_host, values

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [5, 40, 130])
@pytest.mark.parametrize("E,d", [(4, 96), (4, 416), (4, 1056), (8, 96), (8, 416), (33, 32), (33, 96), (33, 1056), (200, 96)])
def test_empty_slices(E, d, T):
    K = 3
    cfg = wl.MoEConfig("slices", E=E, K=K, d_model=d, d_ff=64, T=T, dtype=wl.BF16, seed=91 + E + d)
    print(f"[E={E} d={d} T={T}]", flush=True)
    Wr = (wl.router_weights(cfg, 0) * np.float32(160.0 / d ** 0.5)).astype(np.float32)
    resident = list(map(int, np.random.default_rng(E * 1000 + d).permutation(E)[:K]))
    e2s = np.full(E, -1, np.int32)
    e2s[resident] = np.arange(K, dtype=np.int32)
    W1, W2 = wl.expert_bank(cfg, 0, resident)
    x = wl.hidden_states(cfg, 0)
    L = b.Layer(E, K, d, 64, T, b.SMOE_BF16, router_w=torch.from_numpy(Wr))
    L.workspace = torch.full((L.workspace.numel() + 4096,), 255, dtype=torch.uint8, device="cuda:0")
    L.rebind()
    d_W1, d_W2, d_x = to_dev(W1), to_dev(W2), to_dev(x)
    for s, e in enumerate(resident):
        L.set_resident(s, e, d_W1[s], d_W2[s])
    ref = oracle.layer_forward(x, Wr, W1, W2, e2s)
    ok = ~ref["ambiguous"]
    for fused in (False, True):
        for t in (L.orig_expert, L.slot, L.orig_gate, L.gate, L.xnorm, L.out):
            t.fill_(-1)
        if fused:
            L.forward_fused(d_x, T, accumulate=0)
        else:
            L.route(d_x, T)
        torch.cuda.synchronize()
        assert np.array_equal(to_host(L.orig_expert)[ok], ref["orig_expert"][ok])
        assert np.array_equal(to_host(L.slot)[ok], ref["slot"][ok])
        np.testing.assert_allclose(to_host(L.orig_gate)[ok], ref["orig_gate"][ok], rtol=1e-5)
        np.testing.assert_allclose(to_host(L.gate)[ok], ref["gate"][ok], rtol=1e-5)
        np.testing.assert_allclose(to_host(L.xnorm), ref["xnorm"], rtol=1e-5)
    assert max_abs_rel(values(to_host(L.out), cfg.dtype)[ok], values(ref["out"], cfg.dtype)[ok]) <= 2e-2
    L.close()


@pytest.mark.parametrize("E,d,T", [(8, 1056, 8193), (8, 2080, 8225), (64, 1056, 8225), (100, 2080, 8193)])
def test_chunks_of_two_token_blocks(E, d, T):
    """More than one staged chunk of x with two token blocks per workgroup (more than 8192 tokens), a last workgroup
    with one token or 33: the router against the oracle."""
    K = min(E, 7)
    cfg = wl.MoEConfig("chunks", E=E, K=K, d_model=d, d_ff=32, T=T, dtype=wl.BF16, seed=E + d)
    print(f"[E={E} d={d} T={T}]", flush=True)
    Wr = (wl.router_weights(cfg, 0) * np.float32(160.0 / d ** 0.5)).astype(np.float32)
    x = wl.hidden_states(cfg, 0)
    e2s = np.full(E, -1, np.int32)
    e2s[:K] = np.arange(K, dtype=np.int32)
    L = b.Layer(E, K, d, 32, T, b.SMOE_BF16, router_w=torch.from_numpy(Wr))
    w1, w2 = (torch.zeros(n, dtype=torch.int16, device="cuda:0") for n in (d * 32, d * 32))
    for s in range(K):
        L.set_resident(s, s, w1, w2)
    ref = oracle.route(x, Wr, e2s, 0)
    ok = ~ref["ambiguous"]
    L.route(to_dev(x), T)
    torch.cuda.synchronize()
    assert np.array_equal(to_host(L.orig_expert)[ok], ref["orig_expert"][ok])
    assert np.array_equal(to_host(L.slot)[ok], ref["slot"][ok])
    np.testing.assert_allclose(to_host(L.orig_gate)[ok], ref["orig_gate"][ok], rtol=1e-5)
    np.testing.assert_allclose(to_host(L.gate)[ok], ref["gate"][ok], rtol=1e-5)
    np.testing.assert_allclose(to_host(L.xnorm), ref["xnorm"], rtol=1e-5)
    L.close()
