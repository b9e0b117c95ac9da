"""Sparse attention with 32-row query blocks on both sides of the rule that picks its form (shared double buffers for launches
that leave compute units with two work-groups or fewer, private halves otherwise), with lists of 1 to all blocks."""
import pytest
import torch

import oracle
import paper_2509_24014_amd as sd
from parity_utils import assert_output_close

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Hq,Hkv,bk,L", [
    (16, 4, 32, 1024), (17, 17, 32, 1024),               # 512 work-groups and the first launch beyond
    (20, 4, 32, 870), (20, 4, 64, 870), (20, 4, 64, 896),    # 560, with and without a partial last block
    (20, 4, 128, 896), (20, 4, 128, 850), (20, 4, 128, 790), # the last 128-key block one tile, one and a bit, a bit
    (40, 8, 64, 420), (2, 2, 64, 1300),                      # 560 with short lists; 82 with lists of up to 21 tiles
])
def test_both_forms(Hq, Hkv, bk, L, D):
    bq, nqb, nkb = 32, -(-L // 32), -(-L // bk)
    g = torch.Generator().manual_seed(L + bk + D)
    q, k, v = ((torch.randn(1, h, L, D, generator=g) * s).to(torch.bfloat16) for h, s in ((Hq, 0.6), (Hkv, 0.6), (Hkv, 1.0)))
    ptr = torch.zeros(1, Hq, nqb + 1, dtype=torch.int32)
    col = torch.zeros(1, Hq, nqb * nkb, dtype=torch.int32)
    for h in range(Hq):   # query block i of head h keeps 1 + (7 h + i) % nkb blocks, every other one the last of the sequence
        at = 0
        for i in range(nqb):
            pick = torch.randperm(nkb, generator=g)[:1 + (7 * h + i) % nkb].tolist()
            if i % 2 == 0 and nkb - 1 not in pick:
                pick[0] = nkb - 1
            col[0, h, at:at + len(pick)] = torch.tensor(sorted(pick), dtype=torch.int32)
            at += len(pick)
            ptr[0, h, i + 1] = at
    want = oracle.attn_sparse(q, k, v, ptr.numpy(), col.numpy(), bq, bk)
    used = int(ptr[0, :, -1].max())
    qd, kd, vd = (t.to(DEV) for t in (q, k, v))
    for cap in {used, nqb * nkb}:   # a capacity that is (nearly) exact and one that promises long lists
        ix = sd.BlockIndex(ptr.to(DEV), col[..., :cap].contiguous().to(DEV), bq, bk, nkb)
        sd.index_validate(ix)
        guard = torch.full((1, Hq, L + 40, D), 7.0, dtype=torch.bfloat16, device=DEV)
        out = sd.attn_sparse(qd, kd, vd, ix, out=guard[:, :, :L])
        assert (guard[:, :, L:] == 7.0).all()
        assert_output_close(out, want, torch.bfloat16, f"32x{bk} L={L} cap={cap}")
