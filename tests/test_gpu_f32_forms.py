"""The forms of the fp32 kernels that short inputs do not reach: work-groups of four waves (more than 256 work-groups), waves
that walk many key tiles, and pooling over more than one segment of 512 key blocks."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2509_24014_amd as sd
from parity_utils import assert_output_close, compare_index, random_csr

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _qkv(B, Hq, Hkv, L, D, seed, scale=0.6):
    g = torch.Generator().manual_seed(seed)
    return [torch.randn(B, h, L, D, generator=g) * s for h, s in ((Hq, scale), (Hkv, scale), (Hkv, 1.0))]


@pytest.mark.parametrize("Hq,Hkv,L,D", [
    (8, 8, 1100, 64),     # 280 work-groups, 35 tiles over four waves, the last one 12 keys
    (8, 2, 1100, 128),
    (16, 4, 544, 128),    # 272 work-groups, whole tiles
    (8, 8, 1025, 64),     # 264, the last tile one key and the last query tile one row
    (8, 8, 1024, 128),    # 256 work-groups: the largest grid of the eight-wave form, four tiles a wave
])
def test_dense_and_statistics(Hq, Hkv, L, D):
    q, k, v = _qkv(1, Hq, Hkv, L, D, seed=L + D)
    qd, kd, vd = (t.to(DEV) for t in (q, k, v))
    guard = torch.full((1, Hq, L + 40, D), 7.0, device=DEV)
    lse = torch.full((1, Hq, L), float("nan"), device=DEV)
    out = sd.attn_dense(qd, kd, vd, out=guard[:, :, :L], lse_out=lse)
    assert (guard[:, :, L:] == 7.0).all()
    assert_output_close(out, oracle.attn_dense(q, k, v), torch.float32, f"dense f32 L={L}")
    want = torch.logsumexp(q.double() @ k.double().repeat_interleave(Hq // Hkv, 1).transpose(-1, -2) / math.sqrt(D), dim=-1)
    assert (lse.cpu().double() - want).abs().max() < 2e-5
    # selection with its own statistics pass, against the oracle
    bq, bk, rho = 64, 64, 0.2
    nkb = -(-L // bk)
    pooled = torch.full((1, Hq, -(-L // bq), nkb), float("nan"), device=DEV)
    ix = sd.select_pattern(qd, kd, bq, bk, rho, pooled_out=pooled)
    sd.index_validate(ix)
    _, col_idx, apool, _ = oracle.select_pattern(q, k, bq, bk, rho)
    # a pooled score is a mean of exp2 of arguments of up to 20 octaves or so, carried to 2^-24 of that: 1.2e-6 and the sums
    assert (np.abs(pooled.cpu().double().numpy() - apool) / apool).max() < 5e-6
    compare_index(ix.col_idx.cpu().numpy(), col_idx, apool.reshape(-1, nkb), oracle.kept_blocks(rho, nkb))


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("bq,bk,L", [(32, 32, 1100), (64, 64, 1100), (128, 128, 1100), (32, 128, 1056), (128, 64, 1056)])
def test_sparse_lists_of_any_length(bq, bk, L, D):
    """Four-wave work-groups on lists of 0 blocks, one block and so on up to all of them, with and without the partial last
    block."""
    H, nqb, nkb = 8, -(-L // bq), -(-L // bk)
    q, k, v = _qkv(1, H, 4, L, D, seed=L + bq + bk)
    rp, ci = random_csr(1, H, nqb, nkb, nkb, seed=bk + D, device="cpu")
    rows = (rp[..., 1:] - rp[..., :-1]).flatten()
    assert rows.min() == 0 and (rows == 1).any() and rows.max() >= nkb - 1
    ix = sd.BlockIndex(rp.to(DEV), ci.to(DEV), bq, bk, nkb)
    sd.index_validate(ix)
    guard = torch.full((1, H, L + 40, D), 7.0, device=DEV)
    out = sd.attn_sparse(q.to(DEV), k.to(DEV), v.to(DEV), ix, out=guard[:, :, :L])
    assert (guard[:, :, L:] == 7.0).all()
    assert_output_close(out, oracle.attn_sparse(q, k, v, rp.numpy(), ci.numpy(), bq, bk), torch.float32, f"sparse f32 {bq}x{bk} L={L}")


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("H,bq,bk,L,longest", [
    (110, 32, 32, 600, 3),     # 2090 work-groups, 3 tiles on average: four waves a list, some without a tile
    (110, 64, 64, 590, 2),     # the same with two-tile blocks, the last one partial (14 keys)
    (110, 128, 32, 600, 4),    # rows of a 128-row query block in four work-groups
    (54, 32, 32, 600, 3),      # 1026
    (40, 32, 32, 600, 3),      # 760
    (40, 32, 64, 600, 6),      # 760, 8 tiles
    (40, 64, 128, 530, 3),     # 680, four-tile blocks, the last one 18 keys
    (64, 32, 32, 1024, 1),     # 2048, at most one tile: one wave a list
    (62, 32, 32, 1010, 4),     # 1984, 3 tiles on average, the last one 18 keys: one wave
    (62, 64, 32, 1000, 3),     # the same with two work-groups a query block
    (62, 128, 64, 1010, 1),    # and with four, two-tile blocks
    (62, 64, 64, 1010, 3),     # 5 tiles on average: two waves
    (62, 128, 128, 1010, 1),   # one four-tile block, the last one 114 keys: two waves
])
def test_sparse_short_lists_on_many_work_groups(H, bq, bk, L, longest, D):
    """The number of waves that split a list follows from the work-groups and the capacity of the lists."""
    nqb, nkb = -(-L // bq), -(-L // bk)
    q, k, v = _qkv(1, H, H // 2, L, D, seed=L + bk + D)
    rp, ci = random_csr(1, H, nqb, nkb, longest, seed=H + bk, device="cpu")
    ci = ci[..., :int(rp[..., -1].max())].contiguous()   # an exact capacity (for the head with the most entries)
    ix = sd.BlockIndex(rp.to(DEV), ci.to(DEV), bq, bk, nkb)
    sd.index_validate(ix)
    guard = torch.full((1, H, L + 40, D), 7.0, device=DEV)
    out = sd.attn_sparse(q.to(DEV), k.to(DEV), v.to(DEV), ix, out=guard[:, :, :L])
    assert (guard[:, :, L:] == 7.0).all()
    assert_output_close(out, oracle.attn_sparse(q, k, v, rp.numpy(), ci.numpy(), bq, bk), torch.float32, f"sparse f32 {bq}x{bk} H={H}")


@pytest.mark.parametrize("bq,L", [(32, 16500), (64, 16500), (128, 16500), (64, 16384), (128, 32800)])
def test_pooling_over_segments(bq, L):
    """516, 512 and 1025 key blocks of 32: one segment filled exactly, a few blocks of a second one, one block of a third."""
    bk, rho, D = 32, 0.1, 64
    q, k, _ = _qkv(1, 1, 1, L, D, seed=L + bq)
    nqb, nkb = -(-L // bq), -(-L // bk)
    pooled = torch.full((1, 1, nqb, nkb), float("nan"), device=DEV)
    ix = sd.select_pattern(q.to(DEV), k.to(DEV), bq, bk, rho, pooled_out=pooled)
    sd.index_validate(ix)
    got, keep = pooled.cpu().double().numpy()[0, 0], oracle.kept_blocks(rho, nkb)
    # every row: finite, and its probabilities add up to one (means of fp32 sums, each to a few 1e-7: well inside 1e-5)
    keys = np.minimum(bk, L - np.arange(nkb) * bk)
    assert np.abs((got * keys).sum(1) - 1.0).max() < 1e-5
    cols = ix.col_idx.cpu().numpy()[0, 0].reshape(nqb, keep)
    for I in (0, nqb // 2, nqb - 1):
        apool = oracle.pool_scores_rows(q, k, bq, bk, 0, 0, I, I + 1)
        assert (np.abs(got[I] - apool[0]) / apool[0]).max() < 5e-6
        want = np.sort(np.argsort(-apool[0], kind="stable")[:keep])
        compare_index(cols[I], want, apool, keep)
