"""smoe_permute and smoe_permute_static on both sides of the batch sizes where the number of launches
changes (2048 and 65536 tokens), at the edges of their 64- and 1024-token blocks, for slot counts
around a wavefront.  Skewed slots, some empty; exact against the oracle's stable sort."""
import numpy as np
import pytest
import torch

import oracle
from paper_2308_15030_amd import binding as b
from harness import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 63, 64, 65, 1024, 2047, 2048, 2049, 3073, 65536, 65537])
@pytest.mark.parametrize("K", [1, 63, 65, 200])
def test_permute_sizes(T, K):
    rng = np.random.default_rng(T * 1000 + K)
    slot = np.minimum((rng.random(T) ** 3 * K).astype(np.int32), K - 1)
    x = rng.integers(0, 1 << 16, (T, 32)).astype(np.uint16)
    xp, perm, inv, off = oracle.permute(x, slot, K)
    L = b.Layer(256, K, 32, 32, T, b.SMOE_BF16)
    L.slot.copy_(to_dev(slot))
    d_x = to_dev(x)
    for static in (False, True):
        if static and T > 65536:
            break
        for t in (L.x_perm, L.perm, L.inv_perm, L.offsets):
            t.fill_(-1)
        if static:
            b.smoe_permute_static(L.handle, d_x, L.slot, T, L.x_perm, L.perm, L.inv_perm, L.offsets)
        else:
            L.permute(d_x, T)
        torch.cuda.synchronize()
        assert np.array_equal(to_host(L.offsets), off)
        assert np.array_equal(to_host(L.perm), perm) and np.array_equal(to_host(L.inv_perm), inv)
        assert np.array_equal(to_host(L.x_perm), xp)
    L.close()


# rows of 4 KB and more (moved by more workgroups up to 8192 tokens), 64 MB of rows and one row more, 32768 tokens and one more
@pytest.mark.parametrize("T,d", [(1, 2048), (63, 2048), (65, 4096), (2049, 2048), (8192, 2080), (8193, 2048), (8192, 4096),
                                 (8193, 4096), (32768, 32), (32769, 32)])
def test_permute_wide_rows(T, d):
    K = 65
    rng = np.random.default_rng(T + d)
    slot = np.minimum((rng.random(T) ** 3 * K).astype(np.int32), K - 1)
    _, perm, inv, off = oracle.permute(None, slot, K)
    x = torch.randint(-32768, 32767, (T, d), dtype=torch.int16, device="cuda:0", generator=torch.Generator("cuda:0").manual_seed(T))
    L = b.Layer(256, K, d, 32, T, b.SMOE_BF16)
    L.slot.copy_(to_dev(slot))
    for static in (False, True):
        for t in (L.x_perm, L.perm, L.inv_perm, L.offsets):
            t.fill_(-1)
        if static:
            b.smoe_permute_static(L.handle, x, L.slot, T, L.x_perm, L.perm, L.inv_perm, L.offsets)
        else:
            L.permute(x, T)
        torch.cuda.synchronize()
        assert np.array_equal(to_host(L.offsets), off)
        assert np.array_equal(to_host(L.perm), perm) and np.array_equal(to_host(L.inv_perm), inv)
        assert torch.equal(L.x_perm.view(torch.int16), x[L.perm.long()])
    L.close()
