"""The two-launch path of smoe_forward for small batches and the router at the edges of its
instances: token blocks (32, 64, 128), expert blocks (32, 64, 128, 256), the largest batch whose
rows fit the LDS and the next one, d_model past one staged chunk.  Each case: choices and outputs
against the oracle, every output bit for bit against the five separate calls, twice accumulated."""
import numpy as np
import pytest
import torch

import oracle
from paper_2308_15030_amd import workloads as wl
from harness import Case, max_abs_rel, to_dev, to_host, values

pytestmark = pytest.mark.gpu

NAMES = ("orig_expert", "orig_gate", "slot", "gate", "xnorm", "count", "gsum", "score", "perm", "inv_perm",
         "offsets", "out")

#        E    K   d_model d_ff  T
SHAPES = [(33, 5, 64, 96, 31), (32, 5, 64, 96, 32), (33, 5, 64, 96, 33),
          (64, 16, 96, 224, 64), (65, 16, 96, 224, 65), (128, 30, 128, 256, 128), (129, 9, 64, 96, 127),
          (256, 20, 32, 64, 129), (200, 40, 32, 64, 2),
          (8, 2, 768, 256, 104), (8, 2, 768, 256, 105),       # last batch that fits the LDS at this width, and the next
          (8, 1, 160, 96, 100),                               # one slot holds every token: four column blocks
          (16, 3, 1056, 64, 40),                              # two staged chunks of x in the router
          (4, 2, 2560, 64, 31), (4, 2, 2560, 64, 32)]         # the second does not fit: router, ranking and sorted tiles


@pytest.mark.parametrize("E,K,d,f,T", SHAPES)
def test_small_batch_edges(E, K, d, f, T):
    cfg = wl.MoEConfig("small", E=E, K=K, d_model=d, d_ff=f, T=T, dtype=wl.BF16, seed=77 + E + T)
    resident = list(map(int, np.random.default_rng(E * 1000 + T).permutation(E)[:K]))
    print(f"[E={E} K={K} d={d} f={f} T={T}]", flush=True)
    # logits of about the same size at every width: the gates are compared at 1e-5
    c = Case(cfg, resident=resident, router_scale=160.0 / d ** 0.5, gate_mode=(E + T) % 2)
    L = c.L
    ref = oracle.layer_forward(c.x, c.Wr, *c.slot_weights_host(), c.e2s, c.gate_mode, residual=c.x)
    res = to_dev(c.x)
    out = L.forward_fused(c.d_x, T, accumulate=0, residual=res)
    L.forward_fused(c.d_x, T, accumulate=1, residual=res)
    torch.cuda.synchronize()
    ok = ~ref["ambiguous"]
    assert np.array_equal(to_host(L.orig_expert)[ok], ref["orig_expert"][ok])
    assert np.array_equal(to_host(L.slot)[ok], ref["slot"][ok])
    np.testing.assert_allclose(to_host(L.orig_gate)[ok], ref["orig_gate"][ok], rtol=1e-5)
    np.testing.assert_allclose(to_host(L.gate)[ok], ref["gate"][ok], rtol=1e-5)
    np.testing.assert_allclose(to_host(L.xnorm), ref["xnorm"], rtol=1e-5)
    assert max_abs_rel(values(to_host(out), cfg.dtype)[ok], values(ref["out"], cfg.dtype)[ok]) <= 2e-2
    _, perm, inv, off = oracle.permute(None, to_host(L.slot), K)
    assert np.array_equal(to_host(L.perm), perm) and np.array_equal(to_host(L.inv_perm), inv)
    assert np.array_equal(to_host(L.offsets), off)
    assert int(to_host(L.count).sum()) == 2 * T
    got = {n: to_host(getattr(L, n)).copy() for n in NAMES}
    for n in NAMES:
        getattr(L, n).fill_(0)
    L.forward(c.d_x, T, accumulate=0, residual=res)
    L.forward(c.d_x, T, accumulate=1, residual=res)
    torch.cuda.synchronize()
    for n in NAMES:
        assert np.array_equal(to_host(getattr(L, n)), got[n]), n
    L.close()
