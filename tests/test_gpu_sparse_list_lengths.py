"""Sparse attention with small query blocks at every short list length: the pipeline copies one to three tiles ahead, so
lists of 1 to 14 tiles, odd and even, whole and with a partial last block, take different numbers of steady and last steps."""
import pytest
import torch

import oracle
import paper_2509_24014_amd as sd
from parity_utils import assert_output_close

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("bq,bk,L", [(64, 64, 896), (64, 64, 870), (64, 32, 450), (64, 128, 1792), (64, 128, 1700), (64, 128, 1750),
                                     (32, 64, 870), (32, 32, 448), (32, 128, 1700)])
def test_lists_of_every_length(bq, bk, L, D):
    g = torch.Generator().manual_seed(L + bq + D)
    q, k, v = ((torch.randn(1, 2, L, D, generator=g) * s).to(torch.bfloat16) for s in (0.6, 0.6, 1.0))
    nqb, nkb = -(-L // bq), -(-L // bk)
    rows, row_ptr = [], [0]
    for i in range(2 * nqb):   # query block i keeps 1 + i % nkb blocks, every other one the last block of the sequence
        keep = 1 + i % nkb
        pick = torch.randperm(nkb, generator=g)[:keep].tolist()
        if i % 2 == 0 and nkb - 1 not in pick:
            pick[0] = nkb - 1
        rows.append(sorted(pick))
    col = torch.zeros(1, 2, nqb * nkb, dtype=torch.int32)
    ptr = torch.zeros(1, 2, nqb + 1, dtype=torch.int32)
    for h in range(2):
        at = 0
        for i in range(nqb):
            r = rows[h * nqb + i]
            col[0, h, at:at + len(r)] = torch.tensor(r, dtype=torch.int32)
            at += len(r)
            ptr[0, h, i + 1] = at
    ix = sd.BlockIndex(ptr.to(DEV), col.to(DEV), bq, bk, nkb)
    sd.index_validate(ix)
    guard = torch.full((1, 2, L + 72, D), 7.0, dtype=torch.bfloat16, device=DEV)
    out = sd.attn_sparse(q.to(DEV), k.to(DEV), v.to(DEV), ix, out=guard[:, :, :L])
    assert (guard[:, :, L:] == 7.0).all()
    assert_output_close(out, oracle.attn_sparse(q, k, v, ptr.numpy(), col.numpy(), bq, bk), torch.bfloat16, f"{bq}x{bk} L={L}")
