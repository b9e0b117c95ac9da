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
