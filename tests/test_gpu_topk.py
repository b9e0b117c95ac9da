"""The kept blocks against a ranking, on the host, of the very pooled scores the selection returned (so: exactly), at row
lengths on both sides of every register form of the top-k kernel and of the one that keeps the row in LDS."""
import numpy as np
import pytest
import torch

import oracle
import paper_2509_24014_amd as sd

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _ranked(scores, keep):
    return np.sort(np.argsort(-scores, kind="stable")[:keep])   # ties: the lower block


@pytest.mark.parametrize("nkb", [1, 63, 64, 65, 128, 129, 256, 257, 512, 513, 1024, 1025])
@pytest.mark.parametrize("rho,split", [(0.3, None), (0.05, 0.6), (1.0, 0.5)])
def test_kept_blocks_are_the_highest_scores(nkb, rho, split):
    L, bq, bk = nkb * 32 - 5, 128, 32
    g = torch.Generator().manual_seed(nkb)
    q = (torch.randn(1, 1, L, 64, generator=g) * 0.6).to(torch.bfloat16).to(DEV)
    k = (torch.randn(1, 1, L, 64, generator=g) * 0.6).to(torch.bfloat16)
    k[:, :, :L // 2 // 32 * 32] = k[:, :, :32].repeat(1, 1, L // 2 // 32, 1)   # equal blocks: exact ties in every row
    k = k.to(DEV)
    pooled = torch.empty(1, 1, -(-L // bq), nkb, device=DEV)
    p = nkb if split is None else int(split * nkb)
    if split is None:
        ix = sd.select_pattern(q, k, bq, bk, rho, pooled_out=pooled)
    else:
        ix = sd.select_pattern_isolated(q, k, bq, bk, rho, p, pooled_out=pooled)
    sd.index_validate(ix)
    keep_lo, keep_hi = oracle.kept_blocks(rho, p) if p else 0, oracle.kept_blocks(rho, nkb - p) if nkb > p else 0
    row_ptr, col = ix.row_ptr.cpu().numpy()[0, 0], ix.col_idx.cpu().numpy()[0, 0]
    for i, scores in enumerate(pooled.cpu().numpy()[0, 0]):
        want = np.concatenate([_ranked(scores[:p], keep_lo), p + _ranked(scores[p:], keep_hi)])
        np.testing.assert_array_equal(col[row_ptr[i]:row_ptr[i + 1]], want)
