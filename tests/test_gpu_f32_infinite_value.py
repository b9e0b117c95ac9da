"""fp32 sparse attention over a key block whose last 32-key tiles lie past the end of the sequence: they hold no key and add
nothing, also where the last row of V that exists is infinite."""
import math

import pytest
import torch

import paper_2509_24014_amd as sd

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("L,bk", [(96, 64), (160, 128), (192, 128), (224, 128)])   # 1, 3, 2, 1 tiles past the end
def test_tiles_past_the_end_add_nothing_to_an_infinite_row(L, bk, D):
    g = torch.Generator().manual_seed(L + bk)
    q, k, v = (torch.randn(1, 1, L, D, generator=g) * s for s in (0.5, 0.5, 1.0))
    v[..., L - 1, 0], v[..., L - 1, 1] = math.inf, -math.inf
    nqb, nkb = -(-L // 32), -(-L // bk)
    ix = sd.BlockIndex((torch.arange(nqb + 1, dtype=torch.int32) * nkb).view(1, 1, -1).to(DEV),
                       torch.arange(nkb, dtype=torch.int32).repeat(nqb).view(1, 1, -1).to(DEV), 32, bk, nkb)
    out = sd.attn_sparse(q.to(DEV), k.to(DEV), v.to(DEV), ix).cpu()
    assert (out[..., 0] == math.inf).all() and (out[..., 1] == -math.inf).all()
    p = torch.softmax(q.double() @ k.double().transpose(2, 3) / math.sqrt(D), dim=3)
    want = p @ v.double().nan_to_num(posinf=0.0, neginf=0.0)
    assert (out[..., 2:] - want[..., 2:]).abs().max() < 1e-5


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("L,stride", [(5, 2**27 - 64), (17, 2**25 - 64)])
def test_rows_far_apart_with_anything_between_them(L, stride, D):
    """Rows half a GB or 128 MB apart: the offsets of rows past the end wrap around 32 bits and land between those that exist."""
    store = torch.full(((L - 1) * stride + D,), math.nan, device=DEV)
    far = store.as_strided((1, 1, L, D), (store.numel() // 4 * 4, store.numel() // 4 * 4, stride, 1))
    g = torch.Generator().manual_seed(L)
    q, k, v = (torch.randn(1, 1, L, D, generator=g).to(DEV) for _ in range(3))
    want = torch.softmax(q.double() @ k.double().transpose(2, 3).contiguous() / math.sqrt(D), dim=3)
    for which in range(2):
        far.copy_(v if which else k)
        kk, vv = (k, far) if which else (far, v)
        ix = sd.BlockIndex(torch.tensor([[[0, 1]]], dtype=torch.int32, device=DEV), torch.zeros(1, 1, 1, dtype=torch.int32, device=DEV), 128, 128, 1)
        pooled = torch.zeros(1, 1, 1, 1, device=DEV)
        for out in (sd.attn_dense(q, kk, vv), sd.attn_sparse(q, kk, vv, ix), sd.attn_dense_select(q, kk, vv, 128, 128, 1.0, pooled_out=pooled)[0]):
            assert (out.double() - want @ v.double()).abs().max() < 1e-5
        assert abs(pooled.item() * L - 1) < 1e-5
        pooled.zero_()
        sd.select_pattern(q, kk, 128, 128, 1.0, pooled_out=pooled)
        assert abs(pooled.item() * L - 1) < 1e-5
