"""Dense and sparse bf16 calls with too few rows to fill the chip, whose keys are split over the waves of a work-group: every form
that the launch rule picks (4 rows groups x 2 parts, 2 x 2, 2 x 4, 1 x 4), at the sizes where it changes, with tails of every
kind and lists that leave some of the tile streams without a tile."""
import math

import pytest
import torch

import paper_2509_24014_amd as sd

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# bf16 inputs, fp32 sums: the probabilities and the output are rounded to bf16 once each, 2^-8 of values up to about 4
MAX, MEAN = 2e-2, 2e-3


def _qkv(B, Hq, Hkv, L, D, seed):
    g = torch.Generator().manual_seed(seed)
    return [torch.randn(B, h, L, D, generator=g).bfloat16() for h in (Hq, Hkv, Hkv)]


def _close(got, want, what):
    d = (got.double().cpu() - want).abs()
    assert torch.isfinite(got).all() and d.max() < MAX and d.mean() < MEAN, f"{what}: {d.max():.3e} {d.mean():.3e}"


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("B,Hq,Hkv,L", [
    (1, 1, 1, 1), (1, 2, 1, 33), (1, 4, 4, 448),    # up to 256 runs of 32 rows, fewer than 8 tiles: 2 x 2
    (1, 4, 2, 449), (1, 1, 1, 8190), (1, 8, 8, 1024),  # from 8 tiles on: 1 x 4, up to 256 runs exactly
    (1, 8, 8, 1025), (1, 32, 32, 500),              # 264 and 512 runs; 17 and 8 tiles: 2 x 4 or 2 x 2 by head dim
    (1, 4, 1, 4090),                                # 512 runs, 64 tiles: 2 x 4
    (1, 27, 27, 600), (1, 32, 8, 1024),             # 513 and 1024 runs: 4 x 2
    (1, 33, 33, 1000), (2, 41, 41, 65),             # 1056 runs: the general kernel; 246 runs
])
def test_dense(B, Hq, Hkv, L, D):
    q, k, v = _qkv(B, Hq, Hkv, L, D, seed=L + D + Hq)
    guard = torch.full((B, Hq, L + 40, D), 7.0, device=DEV, dtype=torch.bfloat16)
    lse = torch.full((B, Hq, L), float("nan"), device=DEV)
    out = sd.attn_dense(q.to(DEV), k.to(DEV), v.to(DEV), out=guard[:, :, :L], lse_out=lse)
    assert (guard[:, :, L:] == 7.0).all()
    kk, vv = (t.repeat_interleave(Hq // Hkv, 1).double() for t in (k, v))
    for h in sorted({0, Hq // 2, Hq - 1}):
        s = q[:, h].double() @ kk[:, h].transpose(1, 2) / math.sqrt(D)
        _close(out[:, h], torch.softmax(s, 2) @ vv[:, h], f"head {h}")
        assert (lse[:, h].cpu().double() - torch.logsumexp(s, 2)).abs().max() < 1e-5


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("lens", [(700, 1, 333), (64, 700, 65)])
def test_dense_lengths_per_sample(lens, D):
    q, k, v = _qkv(3, 4, 2, 700, D, seed=sum(lens))
    out = torch.full((3, 4, 700, D), 7.0, device=DEV, dtype=torch.bfloat16)
    sd.attn_dense(q.to(DEV), k.to(DEV), v.to(DEV), out=out, seq_lens=torch.tensor(lens, dtype=torch.int32, device=DEV))
    kk, vv = (t.repeat_interleave(2, 1).double() for t in (k, v))
    for b, n in enumerate(lens):
        s = q[b, :, :n].double() @ kk[b, :, :n].transpose(1, 2) / math.sqrt(D)
        _close(out[b, :, :n], torch.softmax(s, 2) @ vv[b, :, :n], f"sample {b}")
        assert (out[b, :, n:] == 7.0).all()


def _random_lists(H, nqb, nkb, longest, seed):
    """Lists of 0, 1, 2, ... blocks up to `longest`, the last block of the sequence in every second one."""
    g = torch.Generator().manual_seed(seed)
    mask = torch.zeros(H, nqb, nkb, dtype=torch.bool)
    for h in range(H):
        for i in range(nqb):
            n = (h + i) % (min(longest, nkb) + 1)
            mask[h, i, torch.randperm(nkb, generator=g)[:n]] = True
            if i % 2 and n:
                mask[h, i, nkb - 1] = True
    count = mask.sum(2)
    row = torch.zeros(1, H, nqb + 1, dtype=torch.int32)
    row[0, :, 1:] = count.cumsum(1)
    col = torch.zeros(1, H, max(int(count.sum(1).max()), 1), dtype=torch.int32)
    for h in range(H):
        idx = mask[h].nonzero()[:, 1]
        col[0, h, :len(idx)] = idx.to(torch.int32)
    return mask, row, col


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("bk", [32, 64, 128])
@pytest.mark.parametrize("H,bq,L,longest", [
    (2, 32, 1100, 9), (2, 32, 1100, 40),       # 70 runs: 1 x 2 or, with longer lists, 1 x 4
    (8, 32, 1990, 40),                         # 504 runs
    (2, 64, 1100, 3), (2, 64, 1100, 40), (8, 64, 1990, 62),
    (2, 128, 1100, 3), (2, 128, 1100, 40),     # rows of a 128-row query block in two or four work-groups
    (8, 128, 1990, 5), (8, 128, 1990, 62),
    (16, 128, 1990, 62), (16, 128, 1990, 4),   # 1008 runs
])
def test_sparse_lists(H, bq, L, longest, bk, D):
    nqb, nkb = -(-L // bq), -(-L // bk)
    q, k, v = _qkv(1, H, H // 2, L, D, seed=L + bk + D + longest)
    k = k * 2   # rows whose logits differ by some tens of octaves from part to part
    mask, row, col = _random_lists(H, nqb, nkb, longest, seed=bq + bk)
    ix = sd.BlockIndex(row.to(DEV), col.to(DEV), bq, bk, nkb)
    sd.index_validate(ix)
    guard = torch.full((1, H, L + 40, D), 7.0, device=DEV, dtype=torch.bfloat16)
    out = sd.attn_sparse(q.to(DEV), k.to(DEV), v.to(DEV), ix, out=guard[:, :, :L])
    assert (guard[:, :, L:] == 7.0).all()
    kk, vv = (t.repeat_interleave(2, 1) for t in (k, v))
    for h in sorted({0, 1, H - 1}):
        m = mask[h].repeat_interleave(bq, 0).repeat_interleave(bk, 1)[:L, :L]
        s = (q[0, h].float() @ kk[0, h].float().t() / math.sqrt(D)).masked_fill(~m, -math.inf)
        _close(out[0, h], (torch.softmax(s, 1).nan_to_num(0.0) @ vv[0, h].float()).double(), f"head {h}")


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("sign", [1, -1])
def test_parts_whose_logits_lie_far_apart(sign, D):
    """Logits that fall or climb along the keys by hundreds of octaves: a part's reference is far from the others', and a stream
    without a tile (rows of one block) must not set one."""
    L, bq, bk, H = 1024, 32, 64, 2
    q, k, v = _qkv(1, H, H, L, D, seed=D)
    q[..., 0] = 8.0
    k[..., 0] = (sign * torch.linspace(-60, 60, L)).bfloat16() - 70.0
    for longest in (1, 16):
        mask, row, col = _random_lists(H, L // bq, L // bk, longest, seed=longest)
        col = torch.cat([col, torch.zeros(1, H, 2000, dtype=torch.int32)], 2)   # a capacity that stands for long lists
        out = sd.attn_sparse(q.to(DEV), k.to(DEV), v.to(DEV), sd.BlockIndex(row.to(DEV), col.to(DEV), bq, bk, L // bk))
        for h in range(H):
            m = mask[h].repeat_interleave(bq, 0).repeat_interleave(bk, 1)
            s = (q[0, h].double() @ k[0, h].double().t() / math.sqrt(D)).masked_fill(~m, -math.inf)
            _close(out[0, h], torch.softmax(s, 1).nan_to_num(0.0) @ v[0, h].double(), f"head {h}")
    out = sd.attn_dense(q.to(DEV), k.to(DEV), v.to(DEV))
    s = q.double() @ k.double().transpose(2, 3) / math.sqrt(D)
    _close(out, torch.softmax(s, 3) @ v.double(), "dense")
