"""Launch shapes that follow from the number of heads and tokens: work-groups of 128 or 256 rows for dense calls of one to a few
rounds of the chip, the switch step of few rows as two kernels, pooling with the keys cut into segments."""
import math

import pytest
import torch

import paper_2509_24014_amd as sd

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
MAX, MEAN = 2e-2, 2e-3   # bf16 outputs of values up to about 4


def _qkv(B, Hq, Hkv, L, D, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return [torch.randn(B, h, L, D, generator=g, device=DEV).bfloat16() for h in (Hq, Hkv, Hkv)]


def _rows(q, k, v, b, h, rows):
    """Attention of some rows of one head in float64: output, log-sum-exp, probabilities."""
    hk = h // (q.shape[1] // k.shape[1])
    s = q[b, h, rows].double() @ k[b, hk].double().t() / math.sqrt(q.shape[3])
    return torch.softmax(s, 1) @ v[b, hk].double(), torch.logsumexp(s, 1), torch.softmax(s, 1)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("B,Hq,Hkv,L", [
    (2, 8, 8, 4500),    # 288 work-groups of 256 rows, 576 of 128: 128
    (1, 8, 2, 6404),    # 208: 256 rows, a partial last tile
    (1, 28, 4, 3776),   # a multiple of 64 and not of 128; 1.64 rounds: 256
    (8, 80, 80, 64),    # one tile of 64 rows
    (8, 40, 40, 100),   # 320 work-groups of 128 rows; of 256 they would be two rounds
    (1, 33, 33, 2300),  # 1.16 rounds
])
def test_dense(B, Hq, Hkv, L, D):
    q, k, v = _qkv(B, Hq, Hkv, L, D, seed=L + D)
    guard = torch.full((B, Hq, L + 20, D), 7.0, device=DEV, dtype=torch.bfloat16)
    lse = torch.full((B, Hq, L), float("nan"), device=DEV)
    out = sd.attn_dense(q, k, v, out=guard[:, :, :L], lse_out=lse)
    assert (guard[:, :, L:] == 7.0).all() and torch.isfinite(out).all() and torch.isfinite(lse).all()
    rows = torch.unique(torch.tensor([0, 31, 63, 64, 127, 128, 255, 256, L // 2, L - 33, L - 2, L - 1], device=DEV).clamp(0, L - 1))
    for b, h in ((0, 0), (B - 1, Hq - 1)):
        want, wl, _ = _rows(q, k, v, b, h, rows)
        d = (out[b, h, rows].double() - want).abs()
        assert d.max() < MAX and d.mean() < MEAN
        assert (lse[b, h, rows].double() - wl).abs().max() < 1e-5


@pytest.mark.parametrize("bq,bk", [(32, 32), (64, 64), (128, 64), (128, 128), (32, 128)])
@pytest.mark.parametrize("B,Hq,Hkv,L,D", [
    (1, 4, 2, 2000, 128),   # two kernels, 14 segments or fewer
    (1, 4, 4, 1000, 64),    # two kernels, four segments
    (1, 1, 1, 705, 128),    # two kernels, the fewest tiles; segments of 256 tokens, the last one 193
    (1, 4, 2, 500, 128),    # one kernel of 128 rows
    (1, 16, 4, 1100, 128),  # one kernel of 256 rows on a part of the chip
    (1, 16, 16, 1030, 64),  # one kernel of 128 rows on a part of the chip
    (1, 40, 40, 1300, 64),  # 1.1 rounds of it
])
def test_switch_step(B, Hq, Hkv, L, D, bq, bk):
    q, k, v = _qkv(B, Hq, Hkv, L, D, seed=L + D + bq)
    nqb, nkb = -(-L // bq), -(-L // bk)
    pooled = torch.full((B, Hq, nqb, nkb), float("nan"), device=DEV)
    lse = torch.full((B, Hq, L), float("nan"), device=DEV)
    out, ix = sd.attn_dense_select(q, k, v, bq, bk, 0.3, pooled_out=pooled, lse_out=lse)
    sd.index_validate(ix)
    keep = sd.kept_blocks(0.3, nkb)
    for h in sorted({0, Hq - 1}):
        want, wl, p = _rows(q, k, v, 0, h, torch.arange(L, device=DEV))
        d = (out[0, h].double() - want).abs()
        assert d.max() < MAX and d.mean() < MEAN
        assert (lse[0, h].double() - wl).abs().max() < 1e-5
        full = torch.zeros(nqb * bq, nkb * bk, dtype=torch.float64, device=DEV)
        full[:L, :L] = p
        count = torch.zeros_like(full)
        count[:L, :L] = 1
        block = lambda x: x.view(nqb, bq, nkb, bk).sum((1, 3))  # noqa: E731
        score = block(full) / block(count)
        # fp32 sums of exponentials whose arguments are carried to 2^-24 of up to 20 octaves
        assert ((pooled[0, h].double() - score).abs() / score).max() < 5e-6
        kth = score.sort(1, descending=True).values[:, keep - 1:keep]
        kept = score.gather(1, ix.col_idx[0, h].view(nqb, keep).long())
        assert (kept >= kth * (1 - 1e-5)).all()


@pytest.mark.parametrize("lens", [(2000, 1, 700), (300, 2000, 1999)])
def test_segments_of_shorter_samples(lens):
    """Per-sample lengths with segments wholly past the end of a sample: scores of the samples are those of each alone."""
    B, H, L, D, bq, bk = 3, 2, 2000, 128, 64, 32
    q, k, v = _qkv(B, H, H, L, D, seed=sum(lens))
    nqb, nkb = -(-L // bq), -(-L // bk)
    pooled = torch.full((B, H, nqb, nkb), 7.0, device=DEV)
    out, ix = sd.attn_dense_select(q, k, v, bq, bk, 0.2, pooled_out=pooled, out=torch.full_like(q, 7.0),
                                   seq_lens=torch.tensor(lens, dtype=torch.int32, device=DEV))
    for b, n in enumerate(lens):
        qb, kb, vb = (t[b:b + 1, :, :n].contiguous() for t in (q, k, v))
        one = torch.empty(1, H, -(-n // bq), -(-n // bk), device=DEV)
        ob, ib = sd.attn_dense_select(qb, kb, vb, bq, bk, 0.2, pooled_out=one)
        got = pooled[b, :, :one.shape[2], :one.shape[3]]
        assert ((got - one[0]).abs() / one[0]).max() < 5e-6
        assert (pooled[b, :, one.shape[2]:] == 7.0).all() and (pooled[b, :, :, one.shape[3]:] == 7.0).all()
        assert (out[b, :, :n].float() - ob[0].float()).abs().max() < MAX and (out[b, :, n:] == 7.0).all()


def test_a_workspace_of_the_smaller_shape_still_serves():
    """The least workspace of the 128-row shape is accepted where 256 rows a work-group would need more; less is refused."""
    B, H, L, D, bq, bk = 1, 16, 1100, 128, 64, 64
    q, k, v = _qkv(B, H, H, L, D, seed=5)
    nqb = nkb = -(-L // 64)
    need = (B * H * nqb * nkb * 4 + 255) // 256 * 256 + B * H * -(-L // 128) * 128 * ((nkb + 1) & ~1) * 4
    want, ix = sd.attn_dense_select(q, k, v, bq, bk, 0.2)
    got, ix2 = sd.attn_dense_select(q, k, v, bq, bk, 0.2, workspace=torch.empty(need, dtype=torch.uint8, device=DEV))
    assert (got.float() - want.float()).abs().max() < MAX
    with pytest.raises(sd.SparsedError):
        sd.attn_dense_select(q, k, v, bq, bk, 0.2, workspace=torch.empty(need - 256, dtype=torch.uint8, device=DEV))


@pytest.mark.parametrize("H,L,D", [(4, 2048, 128), (8, 1000, 128), (4, 1000, 64), (16, 1000, 128), (4, 1000, 128)])
@pytest.mark.parametrize("offset", [0, 14, 100])
def test_scores_of_a_switch_step_as_two_kernels_keep_their_bits(H, L, D, offset):
    """Logits with a common offset of up to 70 (100 octaves): a score is as good as without, where the row statistics go from the one
    kernel to the other as where one kernel does both."""
    q, k, v = _qkv(1, H, H, L, D, seed=L + D)
    q, k = q * 0.5, k * 0.5
    q[..., 0], k[..., 0] = 8, offset / 8 * D ** 0.5 / 1.4426950408889634
    nb = -(-L // 64)
    pooled = torch.zeros(1, H, nb, nb, device=DEV)
    sd.attn_dense_select(q, k, v, 64, 64, 0.2, pooled_out=pooled)
    p = _rows(q, k, v, 0, 0, torch.arange(L, device=DEV))[2]
    pad = lambda x: torch.nn.functional.pad(x, (0, nb * 64 - L, 0, nb * 64 - L)).view(nb, 64, nb, 64).sum((1, 3))  # noqa: E731
    want = pad(p) / pad(torch.ones_like(p))
    # arguments are differences to the row's reference of some ten octaves, of fp32 logits that carry 2^-24 of up to 100 octaves each
    # (an error of its own for every pair, averaged over 4096): 100 * 2^-24 * ln 2 / sqrt(4096) = 6e-8, and the sums' own 1e-7;
    # a reference that were rounded like the logits would be off by 100 * 2^-24 * ln 2 = 4e-6 for a whole row
    error = ((pooled[0, 0].double() - want) / want)[:L // 64, :L // 64]
    assert error.pow(2).mean().sqrt() < 2.5e-7, error.pow(2).mean().sqrt()


@pytest.mark.parametrize("L", [500, 1000])   # one kernel, two
def test_scores_of_rows_with_an_infinite_logit_are_not_numbers(L):
    q, k, v = _qkv(1, 2, 2, L, 128, seed=L)
    q[0, 0] = q[0, 0].abs()
    k[0, 0, 40, 2] = math.inf
    nb = -(-L // 64)
    pooled = torch.zeros(1, 2, nb, nb, device=DEV)
    out, _ = sd.attn_dense_select(q, k, v, 64, 64, 0.2, pooled_out=pooled)
    assert pooled[0, 0].isnan().all() and out[0, 0].isnan().all()
    assert torch.isfinite(pooled[0, 1]).all() and torch.isfinite(out[0, 1]).all()
