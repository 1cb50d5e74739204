"""fp32 layers at the edges of the router's and the expert FFN's instances: widths that end inside a
panel or a reduction step, one to many row tiles per slot, every width of the feature range, expert
counts around 32 / 64 / 128.  Against the oracle, 1e-4 of the tensor's scale as in test_parity_gpu.py."""
import numpy as np
import pytest
import torch

import oracle
from paper_2308_15030_amd import workloads as wl
from harness import Case, max_abs_rel, to_host, values

pytestmark = pytest.mark.gpu

#        E    K  d_model d_ff  T
SHAPES = [(8, 4, 64, 256, 16), (8, 4, 64, 256, 17), (8, 4, 256, 1024, 512), (8, 2, 768, 512, 130), (4, 1, 52, 100, 33),
          (33, 3, 68, 60, 65), (130, 5, 36, 132, 70), (200, 20, 132, 128, 300), (64, 2, 128, 320, 1), (65, 40, 64, 64, 40)]


@pytest.mark.parametrize("E,K,d,f,T", SHAPES)
def test_fp32_edges(E, K, d, f, T):
    cfg = wl.MoEConfig("fp32", E=E, K=K, d_model=d, d_ff=f, T=T, dtype=wl.F32, seed=55 + E + T)
    resident = list(map(int, np.random.default_rng(E * 1000 + T).permutation(E)[:K]))
    print(f"[E={E} K={K} d={d} f={f} T={T}]", flush=True)
    c = Case(cfg, resident=resident, router_scale=160.0 / d ** 0.5, gate_mode=T % 2)
    L = c.L
    ref = oracle.layer_forward(c.x, c.Wr, *c.slot_weights_host(), c.e2s, c.gate_mode, residual=c.x)
    out = L.forward(c.d_x, T, accumulate=0, residual=c.d_x)
    torch.cuda.synchronize()
    ok = ~ref["ambiguous"]
    assert np.array_equal(to_host(L.orig_expert)[ok], ref["orig_expert"][ok])
    assert np.array_equal(to_host(L.slot)[ok], ref["slot"][ok])
    np.testing.assert_allclose(to_host(L.gate)[ok], ref["gate"][ok], rtol=1e-5)
    np.testing.assert_allclose(to_host(L.xnorm), ref["xnorm"], rtol=1e-5)
    if ok.all():
        assert np.array_equal(to_host(L.perm), ref["perm"]) and np.array_equal(to_host(L.inv_perm), ref["inv_perm"])
        for k in range(K):
            a, b = ref["offsets"][k], ref["offsets"][k + 1]
            assert max_abs_rel(to_host(L.y_perm)[a:b].astype(np.float64), ref["y_perm"][a:b]) <= 1e-4, k
    assert max_abs_rel(values(to_host(out), cfg.dtype)[ok], values(ref["out"], cfg.dtype)[ok]) <= 1e-4
    L.close()
