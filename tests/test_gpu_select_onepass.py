"""Pooled scores in one pass over the keys (a selection without handed-over row statistics) at the edges of its parked
columns: they are stored in pairs, or once per two key tiles, and a slab is reused by later units."""
import numpy as np
import pytest
import torch

import oracle
import paper_2509_24014_amd as sd
from parity_utils import compare_index

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("B,Hq,Hkv,L,D,bq,bk", [
    (1, 2, 1, 960, 128, 128, 64),      # an odd number of tiles: the last column has no partner
    (1, 2, 2, 992, 128, 32, 32),       # an odd number of 32-key blocks
    (2, 2, 2, 600, 64, 64, 32),        # last 32-key block 24 keys
    (1, 2, 2, 960, 64, 64, 128),       # the last 128-key block is one tile
    (1, 1, 1, 65, 64, 32, 64),         # one key and one row in the last tile
    (1, 1, 1, 20, 128, 128, 128),      # a single partial tile
    (1, 1, 1, 4100, 128, 64, 64),      # 65 columns: the closing pass goes round more than once, its last group one column
    (3, 400, 200, 140, 64, 128, 64),   # more units than work-groups, the second unit of a head 12 rows
])
def test_pooled_scores_and_index(B, Hq, Hkv, L, D, bq, bk):
    g = torch.Generator().manual_seed(L + bq + bk)
    scale = 0.45 if D == 128 else 0.6
    q, k = ((torch.randn(B, h, L, D, generator=g) * scale).to(torch.bfloat16) for h in (Hq, Hkv))
    nqb, nkb, rho = -(-L // bq), -(-L // bk), 0.3
    pooled = torch.full((B, Hq, nqb, nkb), float("nan"), device=DEV)
    ix = sd.select_pattern(q.to(DEV), k.to(DEV), bq, bk, rho, pooled_out=pooled)
    sd.index_validate(ix)
    row_ptr, col_idx, apool, _ = oracle.select_pattern(q, k, bq, bk, rho)
    rel = np.abs(pooled.cpu().double().numpy() - apool) / apool
    assert rel.max() < 5e-6, f"pooled scores off by {rel.max():.2e} relative"   # the bar of the other pooling kernels
    np.testing.assert_array_equal(ix.row_ptr.cpu().numpy(), row_ptr)
    keep = oracle.kept_blocks(rho, nkb)
    compare_index(ix.col_idx.cpu().numpy()[..., :nqb * keep], col_idx, apool.reshape(-1, nkb), keep)
