"""A padded batch (a length per sample) against the same samples called one by one, with grouped heads: the samples
alternate in launch order, so every (batch, head) slab has to be visited exactly once and be the right one."""
import pytest
import torch

import paper_2509_24014_amd as sd

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype,Hq,Hkv,L,D,lens,bq,bk", [
    (torch.bfloat16, 6, 2, 300, 64, [300, 1, 170], 128, 64),       # groups of three heads; a sample of one token
    (torch.bfloat16, 4, 4, 270, 128, [64, 270, 200, 33], 64, 128),
    (torch.bfloat16, 8, 1, 200, 128, [200, 130], 32, 32),          # one group holds all heads
    (torch.float32, 6, 3, 150, 64, [33, 150, 90], 32, 64),
])
def test_samples_of_a_padded_batch_equal_single_calls(dtype, Hq, Hkv, L, D, lens, bq, bk):
    g = torch.Generator().manual_seed(L + Hq)
    B = len(lens)
    q, k, v = ((torch.randn(B, h, L, D, generator=g) * 0.5).to(dtype).to(DEV) for h in (Hq, Hkv, Hkv))
    sl = torch.tensor(lens, dtype=torch.int32, device=DEV)
    dense = sd.attn_dense(q, k, v, out=torch.zeros_like(q), seq_lens=sl)
    nqb, nkb = -(-L // bq), -(-L // bk)
    pooled = torch.zeros(B, Hq, nqb, nkb, device=DEV)
    ix = sd.select_pattern(q, k, bq, bk, 0.4, pooled_out=pooled, seq_lens=sl)
    sparse = sd.attn_sparse(q, k, v, ix, out=torch.zeros_like(q), seq_lens=sl)
    # sums of a shorter tensor are grouped differently where its length picks another tile: one rounding of the type
    tol = 2e-2 if dtype == torch.bfloat16 else 1e-5
    for b, n in enumerate(lens):
        q1, k1, v1 = (x[b:b + 1, :, :n].contiguous() for x in (q, k, v))
        torch.testing.assert_close(dense[b:b + 1, :, :n], sd.attn_dense(q1, k1, v1), rtol=tol, atol=tol)
        p1 = torch.zeros(1, Hq, -(-n // bq), -(-n // bk), device=DEV)
        ix1 = sd.select_pattern(q1, k1, bq, bk, 0.4, pooled_out=p1)
        torch.testing.assert_close(pooled[b:b + 1, :, :p1.shape[2], :p1.shape[3]], p1, rtol=5e-6, atol=0)
        assert torch.equal(ix.row_ptr[b, :, :ix1.row_ptr.shape[2]], ix1.row_ptr[0])
        used = ix1.row_ptr[0, 0, -1].item()
        assert torch.equal(ix.col_idx[b, :, :used], ix1.col_idx[0, :, :used])
        torch.testing.assert_close(sparse[b:b + 1, :, :n], sd.attn_sparse(q1, k1, v1, ix1), rtol=tol, atol=tol)
        assert not dense[b, :, n:].any() and not sparse[b, :, n:].any()
