"""A token with a NaN among its hidden states (all its logits are NaN): its slot stays inside [0, K), it
has its place in the order, its row of the output is written and is NaN, and the other tokens' results are
bit for bit those of a batch without it.  Every route of smoe_forward (two launches, sorted tiles) and the
separate calls, bf16 and fp32."""
import numpy as np
import pytest
import torch

from paper_2308_15030_amd import workloads as wl
from harness import Case, to_host, values

pytestmark = pytest.mark.gpu

PER_TOKEN = ("orig_expert", "orig_gate", "slot", "gate", "xnorm")


@pytest.mark.parametrize("dtype,T,fused", [(wl.BF16, 1, True), (wl.BF16, 20, True), (wl.BF16, 100, True), (wl.BF16, 300, True),
                                           (wl.BF16, 20, False), (wl.BF16, 300, False), (wl.F32, 20, False), (wl.F32, 300, False)])
def test_nan_token(dtype, T, fused):
    cfg = wl.MoEConfig("nan", E=40, K=7, d_model=128, d_ff=192, T=T, dtype=dtype, seed=7)
    c = Case(cfg, router_scale=14.0)
    L, K, bad = c.L, cfg.K, T // 2
    runs = []
    for with_nan in (False, True):
        x = c.d_x.clone()
        if with_nan:
            x.view(torch.bfloat16 if dtype == wl.BF16 else torch.float32)[bad, 5] = float("nan")
        for t in (L.slot, L.perm, L.inv_perm, L.out):
            t.fill_(-1)
        (L.forward_fused if fused else L.forward)(x, T, accumulate=0)
        torch.cuda.synchronize()
        runs.append({n: to_host(getattr(L, n)).copy() for n in PER_TOKEN + ("perm", "inv_perm", "offsets", "out")})
    clean, got = runs
    assert 0 <= got["slot"][bad] < K
    assert got["offsets"][K] == T
    assert np.array_equal(np.sort(got["perm"]), np.arange(T)) and np.array_equal(got["perm"][got["inv_perm"]], np.arange(T))
    assert np.isnan(values(got["out"], dtype)[bad]).all()
    rest = np.arange(T) != bad
    for n in PER_TOKEN + ("out",):
        assert np.array_equal(got[n][rest], clean[n][rest]), n
    L.close()
