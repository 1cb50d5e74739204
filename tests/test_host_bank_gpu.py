"""Loads whose source is pinned host memory take a bounded number of workgroups that walk the tiles:
the slot bytes against the documented packed layout, for tile counts below, at and above that number
(64) and with remainders.  Byte-exact."""
import numpy as np
import pytest
import torch

from paper_2308_15030_amd import binding as b

pytestmark = pytest.mark.gpu


def _packed(w, dtype):
    """Slot order of a matrix [R, N]: bf16 MFMA operand blocks, fp32 panels of 64 features."""
    R, N = w.shape
    if dtype == b.SMOE_BF16:                       # [n/32][r/16][(r%16)/8][n%32][r%8]
        return w.reshape(R // 16, 2, 8, N // 32, 32).transpose(3, 0, 1, 4, 2).reshape(-1)
    return np.concatenate([w[:, c:c + 64].reshape(R // 4, 4, -1).transpose(0, 2, 1).reshape(-1)
                           for c in range(0, N, 64)])


def _bank(E, d, f, dtype):
    kind = torch.int16 if dtype == b.SMOE_BF16 else torch.float32
    g = torch.Generator().manual_seed(d * 10007 + f)
    return [torch.randint(-16000, 16000, (E, *s), generator=g).to(kind).pin_memory() for s in ((d, f), (f, d))]


def _slots(L, d, f, kind):
    return [t.reshape(-1).view(kind).cpu().numpy().reshape(-1, d * f) for t in (L.slot_w1, L.slot_w2)]


@pytest.mark.parametrize("dtype,d,f", [
    (b.SMOE_BF16, 32, 32), (b.SMOE_BF16, 256, 256), (b.SMOE_BF16, 256, 288), (b.SMOE_BF16, 416, 1696), (b.SMOE_BF16, 768, 3072),
    (b.SMOE_F32, 4, 8), (b.SMOE_F32, 256, 512), (b.SMOE_F32, 260, 516), (b.SMOE_F32, 252, 1004)])
@pytest.mark.parametrize("device_w2", [False, True])
def test_set_resident_from_pinned(dtype, d, f, device_w2):
    w1, w2 = _bank(3, d, f, dtype)
    s2 = w2.to("cuda:0") if device_w2 else w2
    L = b.Layer(4, 3, d, f, 8, dtype)
    for s in range(3):
        L.set_resident(s, 3 - s, w1[2 - s], s2[2 - s])
    torch.cuda.synchronize()
    got = _slots(L, d, f, w1.dtype)
    for s in range(3):
        for have, w in zip(got, (w1, w2)):
            assert np.array_equal(have[s], _packed(w[2 - s].numpy(), dtype))
    L.close()


@pytest.mark.parametrize("d,f", [(32, 32), (416, 1696)])
def test_update_on_device_from_pinned(d, f):
    E, K = 9, 4
    w1, w2 = _bank(E, d, f, b.SMOE_BF16)
    L = b.Layer(E, K, d, f, 8, b.SMOE_BF16)
    for s in range(K):
        L.set_resident(s, s, w1[s], w2[s])
    L.score.copy_(torch.arange(E, dtype=torch.float32))        # 5 .. 8 are wanted: every slot changes
    L.update_on_device(w1, w2)
    torch.cuda.synchronize()
    s2e = L.maps()[0].tolist()
    assert s2e == [8, 7, 6, 5]
    got = _slots(L, d, f, w1.dtype)
    for s, e in enumerate(s2e):
        for have, w in zip(got, (w1, w2)):
            assert np.array_equal(have[s], _packed(w[e].numpy(), b.SMOE_BF16))
    L.close()
