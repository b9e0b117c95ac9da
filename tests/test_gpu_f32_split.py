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
@pytest.mark.parametrize("H,keep", [(8, 1), (8, 7), (40, 1), (40, 7), (70, 1), (70, 2), (70, 7)])
def test_every_form_of_the_sparse_launch(H, keep, D):
    """240, 1200 and 2100 work-groups with lists of 1 to 14 tiles: one, two, four and eight waves a list."""
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
