"""Ranking and importance of a prefill batch (smoe_forward's second launch) at the edges of their
blocks: 4 and 16 tokens per thread of the importance sums (1024 and 4096 tokens), 1024-token sort
blocks, histogram rows per pass for slot counts that do and do not divide 1024, the router with two
token blocks (more than 8192 tokens).  Positions and counts are exact against the oracle's stable
sort; the sums against 64 bits at 1e-5 (at most 8225 fp32 terms of one sign, added in 256 strands);
every result bit for bit against the separate calls."""
import numpy as np
import pytest
import torch

import oracle
from paper_2308_15030_amd import workloads as wl
from harness import Case, to_host

pytestmark = pytest.mark.gpu

NAMES = ("orig_expert", "orig_gate", "slot", "gate", "xnorm", "count", "gsum", "score", "perm", "inv_perm", "offsets")


@pytest.mark.parametrize("T", [129, 1024, 1025, 4096, 4097, 8192, 8225])
@pytest.mark.parametrize("E,K", [(256, 200), (100, 65), (8, 3), (33, 1)])
def test_rank_importance_edges(T, E, K):
    cfg = wl.MoEConfig("rank", E=E, K=K, d_model=32, d_ff=32, T=T, dtype=wl.BF16, seed=T + E)
    print(f"[T={T} E={E} K={K}]", flush=True)
    c = Case(cfg, resident=list(map(int, np.random.default_rng(T + E).permutation(E)[:K])), router_scale=28.0)
    L = c.L
    L.forward_fused(c.d_x, T, accumulate=0)
    L.forward_fused(c.d_x, T, accumulate=1)
    torch.cuda.synchronize()
    got = {n: to_host(getattr(L, n)).copy() for n in NAMES}
    _, perm, inv, off = oracle.permute(None, got["slot"], K)
    assert np.array_equal(got["perm"], perm) and np.array_equal(got["inv_perm"], inv) and np.array_equal(got["offsets"], off)
    oe = got["orig_expert"]
    assert np.array_equal(got["count"], 2 * np.bincount(oe, minlength=E))
    og, xn = got["orig_gate"].astype(np.float64), got["xnorm"].astype(np.float64)
    np.testing.assert_allclose(got["gsum"], 2 * np.bincount(oe, og, E), rtol=1e-5)
    np.testing.assert_allclose(got["score"], 2 * np.bincount(oe, og * xn, E) * to_host(L.expert_norm), rtol=1e-5)
    for n in NAMES:
        getattr(L, n).fill_(0)
    L.forward(c.d_x, T, accumulate=0)
    L.forward(c.d_x, T, accumulate=1)
    torch.cuda.synchronize()
    for n in NAMES:
        assert np.array_equal(to_host(getattr(L, n)), got[n]), n
    L.close()
