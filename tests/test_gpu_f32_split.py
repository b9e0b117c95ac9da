"""fp32 products on split operands (three bf16 parts a value): inputs whose parts cannot stand for them (infinite, not a number,
beyond the largest bf16 number) give what the fp32 matrix instruction gives, inputs of very different size are carried like any
fp32 number, and every form of the sparse launch agrees with 64 bits."""
import math

import pytest
import torch

import paper_2509_24014_amd as sd

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _qkv(H, L, D, seed):
    g = torch.Generator().manual_seed(seed)
    return [torch.randn(1, H, L, D, generator=g) * s for s in (0.6, 0.6, 1.0)]


def _exact(q, k, v):
    s = q.double() @ k.double().transpose(2, 3) / math.sqrt(q.shape[3])
    return torch.softmax(s, dim=3) @ v.double(), torch.logsumexp(s, dim=3), torch.softmax(s, dim=3)


@pytest.mark.parametrize("H,L,D", [(2, 300, 64), (2, 300, 128), (20, 480, 128), (20, 480, 64)])   # 8 and 4 waves a work-group
def test_values_that_do_not_split(H, L, D):
    q, k, v = _qkv(H, L, D, seed=L + D)
    v[0, 0, 17, 3], v[0, 0, L - 1, 4] = math.inf, -math.inf     # a column each
    v[0, 0, 18, 5] = 3.4e38                                     # rounds to infinity in bf16
    k[0, 1, 40, 2] = -math.inf                                  # logits of -inf and +inf by the sign of q
    q[0, 1, 7, 9] = math.nan                                    # one row
    lse = torch.empty(1, H, L, device=DEV)
    out = sd.attn_dense(q.to(DEV), k.to(DEV), v.to(DEV), lse_out=lse).cpu()
    want, wl, _ = _exact(q, k, v)
    assert (out[0, 0, :, 3] == math.inf).all() and (out[0, 0, :, 4] == -math.inf).all()
    assert torch.allclose(out[0, 0, :, 5].double(), want[0, 0, :, 5], rtol=1e-5)
    rest = [c for c in range(D) if c not in (3, 4, 5)]
    assert (out[0, 0][:, rest] - want[0, 0][:, rest]).abs().max() < 1e-5
    plus = q[0, 1, :, 2] < 0                                    # a logit of +inf: the softmax of the row is not a number
    plus[7] = True
    assert out[0, 1][plus].isnan().all() and lse.cpu()[0, 1][plus].isnan().all()
    assert (out[0, 1][~plus] - want[0, 1][~plus]).abs().max() < 1e-5
    assert (lse.cpu()[0, 1][~plus] - wl[0, 1][~plus]).abs().max() < 1e-5


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("bq", [32, 64, 128])
def test_pooling_with_infinite_keys(bq, D):
    L, bk = 300, 64
    q, k, _ = _qkv(1, L, D, seed=bq + D)
    q = q.abs()
    k[0, 0, 40, 2] = -math.inf                                  # that key's probability is 0 in every row
    lse = torch.logsumexp(q.double() @ k.double().transpose(2, 3) / math.sqrt(D), dim=3).float().to(DEV)
    pooled = torch.full((1, 1, -(-L // bq), 5), float("nan"), device=DEV)
    sd.select_pattern(q.to(DEV), k.to(DEV), bq, bk, 0.5, lse_in=lse.contiguous(), pooled_out=pooled)
    p = torch.softmax(q.double() @ k.double().transpose(2, 3) / math.sqrt(D), dim=3)
    for I in range(-(-L // bq)):
        for J in range(5):
            want = p[0, 0, I * bq:(I + 1) * bq, J * bk:(J + 1) * bk].mean()
            assert abs(pooled[0, 0, I, J].item() - want) < 5e-6 * want


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("H,L", [(1, 33), (2, 700), (24, 700)])
def test_inputs_of_very_different_size(H, L, D):
    """Sums of products whose sizes span twenty octaves. A product of split operands is carried to 3 * 2^-26 of itself and a sum of
    D = 128 of them in 48 roundings, each at most 2^-24 of the sum of magnitudes: logits to 6e-6 of that, outputs likewise."""
    g = torch.Generator().manual_seed(L + D)
    q, k, v = _qkv(H, L, D, seed=L)
    q, k = (x * torch.exp2(torch.randint(-8, 3, x.shape, generator=g).float()) for x in (q, k))
    v = v * torch.exp2(torch.randint(-10, 11, v.shape, generator=g).float())
    out = sd.attn_dense(q.to(DEV), k.to(DEV), v.to(DEV)).cpu().double()
    want, _, p = _exact(q, k, v)
    size = (q.double().abs() @ k.double().abs().transpose(2, 3) / math.sqrt(D)).amax(dim=3, keepdim=True)
    bound = (p @ v.double().abs()) * (2 * 6e-6 * size + 1e-5)
    assert ((out - want).abs() <= bound).all()


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("H,keep", [(8, 1), (8, 7),                           # 240 work-groups: eight waves a list
                                    (40, 1), (40, 7), (70, 2), (70, 7),       # 1200 and 2100: four
                                    (64, 1), (67, 1),                         # 1920 and 2010, two tiles: one
                                    (64, 2), (64, 3), (70, 1)])               # and four, six, 2100 and two: two
def test_every_form_of_the_sparse_launch(H, keep, D):
    """240 to 2100 work-groups with lists of 2 to 14 tiles: one, two, four and eight waves a list."""
    L, bq, bk = 950, 64, 64
    nqb, nkb = 15, 15
    q, k, v = _qkv(H, L, D, seed=H + keep)
    g = torch.Generator().manual_seed(keep)
    sel = torch.rand(1, H, nqb, nkb, generator=g).topk(keep, 3).indices.sort(3).values
    ix = sd.BlockIndex((torch.arange(nqb + 1, dtype=torch.int32) * keep).expand(1, H, nqb + 1).contiguous().to(DEV),
                       sel.to(torch.int32).reshape(1, H, -1).contiguous().to(DEV), bq, bk, nkb)
    out = sd.attn_sparse(q.to(DEV), k.to(DEV), v.to(DEV), ix).cpu()
    mask = torch.zeros(1, H, nqb, nkb, dtype=torch.bool).scatter_(3, sel, True)
    mask = mask.repeat_interleave(bq, 2).repeat_interleave(bk, 3)[:, :, :L, :L]
    s = (q @ k.transpose(2, 3)).double() / math.sqrt(D)
    want = torch.softmax(s.masked_fill(~mask, -math.inf), dim=3) @ v.double()
    assert (out - want).abs().max() < 1e-5


def _sparse_index(H, L, keep, seed):
    n = -(-L // 64)
    sel = torch.rand(1, H, n, n, generator=torch.Generator().manual_seed(seed)).topk(keep, 3).indices.sort(3).values
    ix = sd.BlockIndex((torch.arange(n + 1, dtype=torch.int32) * keep).expand(1, H, n + 1).contiguous().to(DEV),
                       sel.to(torch.int32).reshape(1, H, -1).contiguous().to(DEV), 64, 64, n)
    mask = torch.zeros(1, H, n, n, dtype=torch.bool).scatter_(3, sel, True)
    return ix, mask.repeat_interleave(64, 2).repeat_interleave(64, 3)[:, :, :L, :L]


def _all_calls(q, k, v, keep=3):
    """(output, exact output, sum of the magnitudes in it) of the dense, the dense and selecting and the sparse call."""
    H, L, D = q.shape[1:]
    qd, kd, vd = (t.to(DEV) for t in (q, k, v))
    s = q.double() @ k.double().transpose(2, 3) / math.sqrt(D)
    ix, mask = _sparse_index(H, L, keep, seed=L)
    for got, logits in ((sd.attn_dense(qd, kd, vd), s), (sd.attn_dense_select(qd, kd, vd, 64, 64, 0.3)[0], s),
                        (sd.attn_sparse(qd, kd, vd, ix), s.masked_fill(~mask, -math.inf))):
        p = torch.softmax(logits, dim=3)
        yield got.cpu().double(), p @ v.double(), p @ v.double().abs()


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("H,L,keep", [(2, 300, 3), (20, 480, 3), (70, 480, 1)])   # 8 and 4 waves; with 1050 work-groups the sparse lists
@pytest.mark.parametrize("e", [-95, -112, -118, -124, -130, -140])
def test_small_values_keep_their_bits(e, H, L, keep, D):
    """Values of V far below what three bf16 parts can hold in full (a part ends at 2^-133): to 1e-5 of the sum of magnitudes, as any
    others, or to the resolution of subnormal numbers, 2^-149 (terms relative to sums of up to 2^9, and the result)."""
    q, k, v = _qkv(H, L, D, seed=L + D)
    v = (v * 2.0 ** -64) * 2.0 ** (e + 64)
    for got, want, size in _all_calls(q, k, v, keep):
        assert ((got - want).abs() <= 1e-5 * size + 2.0 ** -147).all()
    v[..., 1::2] = torch.randn(v[..., 1::2].shape, generator=torch.Generator().manual_seed(e))   # beside ordinary columns
    if e >= -118:
        for got, want, size in _all_calls(q, k, v, keep):
            assert ((got - want).abs() <= 1e-5 * size).all()


@pytest.mark.parametrize("H,L,keep", [(2, 300, 3), (20, 480, 8), (5, 2100, 30)])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("e", [-127, -132, -140])
def test_small_columns_beside_ordinary_and_empty_ones(e, H, L, keep, D):
    """A few columns of V below the smallest normal number, at -140 below the smallest part too: their sums are right to the resolution of
    subnormal numbers and not zeros; columns of zeros, more of them in one head, stay zeros."""
    q, k, v = _qkv(H, L, D, seed=L + D)
    v[..., 3::16] = (v[..., 3::16] * 2.0 ** -64) * 2.0 ** (e + 64)
    v[..., 8::16] = 0.0
    v[:, 0, :, 1::2] = 0.0
    for got, want, size in _all_calls(q, k, v, keep):
        assert ((got - want).abs() <= 1e-5 * size + 2.0 ** -147).all()
        assert (got[..., 8::16] == 0).all()
        assert (got[:, 1:, :, 3::16].abs().amax((2, 3)) > 2.0 ** (e - 8)).all()


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("H,L", [(2, 300), (20, 480)])
@pytest.mark.parametrize("e", [100, 112, 120, 125, -112, -125])
def test_logits_of_small_and_large_factors(e, H, L, D):
    q, k, v = _qkv(H, L, D, seed=L + D)
    q, k = q * 2.0 ** -e, k * 2.0 ** e
    for got, want, size in _all_calls(q, k, v):
        assert ((got - want).abs() <= 1e-5 * size).all()
    p = _exact(q, k, v)[2]
    n = -(-L // 64)
    lse = torch.logsumexp(q.double() @ k.double().transpose(2, 3) / math.sqrt(D), dim=3).float().contiguous().to(DEV)
    pooled = torch.zeros(1, H, n, n, device=DEV)
    sd.select_pattern(q.to(DEV), k.to(DEV), 64, 64, 0.3, lse_in=lse, pooled_out=pooled)
    whole = L // 64
    want = p[:, :, :whole * 64, :whole * 64].view(1, H, whole, 64, whole, 64).mean((3, 5))
    assert ((pooled.cpu().double()[:, :, :whole, :whole] - want).abs() <= 5e-6 * want).all()


@pytest.mark.parametrize("octaves,e", [(60, 60), (100, 100), (115, 113), (125, 124), (130, 125), (140, 126)])
@pytest.mark.parametrize("D", [64, 128])
def test_large_values_at_small_probabilities(octaves, e, D):
    """One key far below the others whose values are as far above: its share of the sums is of their size."""
    q, k, v = _qkv(2, 300, D, seed=D)
    q[..., 0], k[..., 0] = 8.0, 0.0
    q[..., 1:], k[..., 1:] = q[..., 1:] * 0.01, k[..., 1:] * 0.01
    k[0, :, 70, 0] = -octaves * math.log(2) * D ** 0.5 / 8
    v[0, :, 70] = 2.0 ** e
    for got, want, size in _all_calls(q, k, v, keep=5):
        # a subnormal probability is a multiple of 2^-149; its logit is carried to 2^-24 of 140 octaves at three roundings
        assert ((got - want).abs() <= 3e-5 * size + 2.0 ** (e - 149)).all()


@pytest.mark.parametrize("D", [64, 128])
def test_columns_and_heads_of_zeros(D):
    q, k, v = _qkv(2, 300, D, seed=D)
    v[..., D // 2:] = 0
    v[:, 1] = 0
    for got, want, size in _all_calls(q, k, v):
        assert not got[..., D // 2:].any() and not got[:, 1].any()
        assert ((got - want).abs() <= 1e-5 * size).all()
