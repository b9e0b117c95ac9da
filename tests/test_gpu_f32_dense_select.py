"""The fp32 dense call that also leaves the pooled scores: every block size and row grouping, partial last blocks on both axes, waves
without a key block, rows whose reference moves while sums are parked, inputs that repeat the work on the fp32 instruction,
lengths at which the sums no longer fit LDS, and lengths per sample."""
import math

import pytest
import torch

import paper_2509_24014_amd as sd

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _check(q, k, v, bq, bk, rho=0.3, lens=None, bar=5e-6, out_bar=1e-5, lse_bar=2e-5):
    B, Hq, L, D = q.shape
    nqb, nkb = -(-L // bq), -(-L // bk)
    qd, kd, vd = (t.to(DEV) for t in (q, k, v))
    guard = torch.full((B, Hq, L + 40, D), 7.0, device=DEV)
    pooled = torch.full((B, Hq, nqb, nkb), 7.0, device=DEV)
    lse = torch.full((B, Hq, L), 7.0, device=DEV)
    sl = None if lens is None else torch.tensor(lens, dtype=torch.int32, device=DEV)
    out, ix = sd.attn_dense_select(qd, kd, vd, bq, bk, rho, out=guard[:, :, :L], lse_out=lse, pooled_out=pooled, seq_lens=sl)
    sd.index_validate(ix)
    assert (guard[:, :, L:] == 7.0).all()
    for b in range(B):
        n = L if lens is None else lens[b]
        nq, nk = -(-n // bq), -(-n // bk)
        kk, vv = (t[b, :, :n].repeat_interleave(Hq // k.shape[1], 0).to(DEV).double() for t in (k, v))
        s = qd[b, :, :n].double() @ kk.transpose(1, 2).contiguous() / math.sqrt(D)
        p = torch.softmax(s, 2)
        assert (out[b, :, :n].double() - p @ vv).abs().max() < out_bar
        assert (lse[b, :, :n].double() - torch.logsumexp(s, 2)).abs().max() < lse_bar
        assert (lse[b, :, n:] == 7.0).all() and (out[b, :, n:] == 7.0).all()
        full, count = (torch.zeros(Hq, nq * bq, nk * bk, dtype=torch.float64, device=DEV) for _ in range(2))
        full[:, :n, :n], count[:, :n, :n] = p, 1
        score = full.view(Hq, nq, bq, nk, bk).sum((2, 4)) / count.view(Hq, nq, bq, nk, bk).sum((2, 4))
        got = pooled[b, :, :nq, :nk].double()
        big = score > 1e-30
        assert ((got - score).abs() / score)[big].max() < bar
        assert got[~big].numel() == 0 or got[~big].max() < 1e-29
        assert (pooled[b, :, nq:] == 7.0).all() and (pooled[b, :, :, nk:] == 7.0).all()
        if lens is None:
            keep = sd.kept_blocks(rho, nk)
            kth = score.sort(2, descending=True).values[..., keep - 1:keep]
            kept = score.gather(2, ix.col_idx[b].view(Hq, nq, keep).long())
            assert (kept >= kth * (1 - 2 * bar)).all()


def _qkv(B, Hq, Hkv, L, D, seed, scale=0.6):
    g = torch.Generator().manual_seed(seed)
    return [torch.randn(B, h, L, D, generator=g) * s for h, s in ((Hq, scale), (Hkv, scale), (Hkv, 1.0))]


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("bq", [32, 64, 128])
@pytest.mark.parametrize("bk", [32, 64, 128])
@pytest.mark.parametrize("H,L", [(2, 33), (3, 700), (10, 1030)])   # fewer key blocks than waves; partial blocks; whole rounds
def test_every_block_size(H, L, bq, bk, D):
    _check(*_qkv(1, H, 1 if H == 3 else H, L, D, seed=L + bq + bk), bq, bk)


@pytest.mark.parametrize("D,bq,H,fit", [(128, 32, 1, 532), (128, 64, 1, 218), (128, 128, 16, 61), (64, 32, 1, 324), (64, 64, 1, 138), (64, 128, 16, 45)])
def test_around_the_blocks_that_fit(D, bq, H, fit):
    """As many key blocks as the LDS holds sums of, and one more (the dense call and a pooling kernel), at head counts for which the
    rule on costs takes the one kernel."""
    for n in (fit, fit + 1):
        _check(*_qkv(1, H, H, 32 * n - 5, D, seed=n), bq, 32, rho=0.05)


@pytest.mark.parametrize("bq,bk", [(32, 32), (64, 128), (128, 64)])
def test_rows_whose_reference_moves(bq, bk):
    """Logits that climb by 200 octaves along the keys: what a wave has parked is relative to references long past."""
    q, k, v = _qkv(1, 4, 4, 900, 64, seed=bq, scale=0.05)
    q[..., 0] = 8.0
    k[..., 0] = torch.linspace(0, 140, 900)
    # logits of up to 140 (200 octaves) are carried to 2^-24 of their size at each of three roundings (the product, the scale, the
    # difference to the reference): 140 * 3 * 2^-24 = 2.5e-5 of a probability, twice that with its normaliser, and of an output of
    # values up to 4 accordingly; a log-sum-exp has that error of its logits and one more rounding: 140 * 4 * 2^-24 = 3.3e-5 on top of its bar
    _check(q, k, v, bq, bk, bar=5e-5, out_bar=2e-4, lse_bar=6e-5)


@pytest.mark.parametrize("bq", [32, 64, 128])
def test_infinite_values(bq):
    L, D, bk = 500, 128, 64
    q, k, v = _qkv(1, 8, 8, L, D, seed=bq)
    clean, _ = sd.attn_dense_select(q.to(DEV), k.to(DEV), v.to(DEV), bq, bk, 0.3)
    v[0, 0, 20, 3] = math.inf
    pooled = [torch.empty(1, 8, -(-L // bq), 8, device=DEV) for _ in range(2)]
    out, _ = sd.attn_dense_select(q.to(DEV), k.to(DEV), v.to(DEV), bq, bk, 0.3, pooled_out=pooled[0])
    v[0, 0, 20, 3] = 0.0
    sd.attn_dense_select(q.to(DEV), k.to(DEV), v.to(DEV), bq, bk, 0.3, pooled_out=pooled[1])
    assert (out[0, 0, :, 3] == math.inf).all()
    rest = [c for c in range(D) if c != 3]
    assert (out[..., rest] - clean[..., rest]).abs().max() < 1e-5
    assert ((pooled[0] - pooled[1]).abs() / pooled[1]).max() < 5e-6


@pytest.mark.parametrize("bq,bk", [(32, 64), (64, 32), (128, 128)])
def test_lengths_per_sample(bq, bk):
    _check(*_qkv(3, 4, 2, 700, 64, seed=bq), bq, bk, lens=[700, 333, 1])


# One wave ranks the row that its work-group has just pooled, with at most 256 work-groups, 256 key blocks and 64 rows a block;
# beyond, a launch of its own does.
@pytest.mark.parametrize("nkb,bq,bk,D", [(1, 32, 32, 64), (2, 128, 128, 128), (63, 32, 32, 64), (64, 64, 32, 128), (65, 32, 32, 128),
                                         (42, 32, 32, 128), (43, 32, 32, 128), (130, 64, 32, 64), (256, 32, 32, 64), (257, 32, 32, 64)])
@pytest.mark.parametrize("rho", [0.05, 0.5, 1.0])
def test_kept_blocks_are_the_highest_of_the_returned_scores(nkb, bq, bk, D, rho):
    L = nkb * bk - 3
    B, H = (3, 2) if nkb < 60 else (1, 1)   # 6 times 42 work-groups rank, 6 times 43 do not; one sample of 256 does
    g = torch.Generator().manual_seed(nkb)
    q, k, v = (torch.randn(B, H, L, D, generator=g).cuda() for _ in range(3))
    if nkb > 2:
        k[:, :, bk:2 * bk] = k[:, :, :bk]   # equal blocks: ties
    nqb = -(-L // bq)
    lens = torch.tensor([L, max(1, L // 2), 1] if B == 3 else [L * 2 // 3], dtype=torch.int32, device="cuda")
    for seq_lens in (None, lens):
        pooled = torch.zeros(B, H, nqb, nkb, dtype=torch.float32, device="cuda")
        index = sd.BlockIndex(torch.full((B, H, nqb + 1), -7, dtype=torch.int32, device="cuda"),
                              torch.full((B, H, nqb * sd.kept_blocks(rho, nkb)), -7, dtype=torch.int32, device="cuda"), bq, bk, nkb)
        sd.attn_dense_select(q, k, v, bq, bk, rho, pooled_out=pooled, index=index, seq_lens=seq_lens)
        rp, ci, scores = index.row_ptr.cpu(), index.col_idx.cpu(), pooled.cpu()
        for b in range(B):
            n = L if seq_lens is None else int(lens[b])
            blocks, rows = -(-n // bk), -(-n // bq)
            keep = sd.kept_blocks(rho, blocks)
            assert rp[b, 0].tolist() == [min(i, rows) * keep for i in range(nqb + 1)]
            assert torch.equal(rp[b], rp[b, :1].expand(H, -1))
            best = torch.sort(-scores[b, :, :rows, :blocks], dim=2, stable=True).indices[..., :keep].sort(dim=2).values
            assert torch.equal(ci[b, :, :rows * keep].view(H, rows, keep).long(), best)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("bq,H", [(64, 2), (128, 40)])   # head counts at which one kernel does both
def test_scores_below_the_smallest_normal_number_are_ranked(bq, H, D):
    """Blocks whose probabilities lie 130 to 146 octaves below the row's largest, the later the larger: their scores are subnormal
    numbers, and the largest of them is kept, not the first."""
    L, bk = 512, 64
    q, k, v = _qkv(1, H, H, L, D, seed=bq + D, scale=0.01)
    q[..., 0], k[..., 0] = 8.0, 0.0
    k[:, :, 256:, 0] = -torch.linspace(146, 130, 256) * math.log(2) * D ** 0.5 / 8
    pooled = torch.zeros(1, H, L // bq, 8, device=DEV)
    _, ix = sd.attn_dense_select(q.to(DEV), k.to(DEV), v.to(DEV), bq, bk, 0.625, pooled_out=pooled)
    p = torch.softmax(q.double() @ k.double().transpose(2, 3) / math.sqrt(D), 3)
    want = p.view(1, H, L // bq, bq, 8, bk).mean((3, 5))
    # a subnormal number is a multiple of 2^-149: the mean is rounded there once, its terms (relative to a row's reference, up to
    # 2^9 times as large) before; and the arguments as in every row
    assert ((pooled.cpu().double() - want).abs() <= 2.0 ** -148 + 2e-3 * want).all()
    assert (want[..., 7] > 2.0 ** -143).all()
    assert (ix.col_idx.cpu().view(1, H, L // bq, 5) == torch.tensor([0, 1, 2, 3, 7])).all()
