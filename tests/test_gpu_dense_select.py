"""GPU parity of the switch step in one call (sparsed_attn_dense_select): output, row log-sum-exp, pooled scores and
index against the fp64 oracle."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2509_24014_amd as sd
from parity_utils import assert_output_close, compare_index

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _qkv(B, Hq, Hkv, L, D, dtype, seed, scale):
    g = torch.Generator().manual_seed(seed)
    return ((torch.randn(B, Hq, L, D, generator=g) * scale).to(dtype), (torch.randn(B, Hkv, L, D, generator=g) * scale).to(dtype),
            torch.randn(B, Hkv, L, D, generator=g).to(dtype))


def _check(q, k, v, bq, bk, rho, views=None):
    B, Hq, L, D = q.shape
    nqb, nkb = -(-L // bq), -(-L // bk)
    qd, kd, vd = views if views is not None else (t.to(DEV) for t in (q, k, v))
    guard = torch.full((B, Hq, L + 72, D), 7.0, dtype=q.dtype, device=DEV)
    pooled = torch.full((B, Hq, nqb, nkb), float("nan"), device=DEV)
    lse = torch.empty(B, Hq, L, device=DEV)
    out, ix = sd.attn_dense_select(qd, kd, vd, bq, bk, rho, out=guard[:, :, :L], lse_out=lse, pooled_out=pooled)
    torch.cuda.synchronize()
    sd.index_validate(ix)
    assert (guard[:, :, L:] == 7.0).all(), "rows past L were written"
    assert_output_close(out, oracle.attn_dense(q, k, v), q.dtype, f"dense+select {bq}x{bk} L={L}")
    row_ptr, col_idx, apool, _ = oracle.select_pattern(q, k, bq, bk, rho)
    rel = np.abs(pooled.cpu().double().numpy() - apool) / apool
    assert rel.max() < 5e-6, f"pooled scores off by {rel.max():.2e} relative"   # the bar of the other pooling kernels
    np.testing.assert_array_equal(ix.row_ptr.cpu().numpy(), row_ptr)
    keep = oracle.kept_blocks(rho, nkb)
    compare_index(ix.col_idx.cpu().numpy()[..., :nqb * keep], col_idx, apool.reshape(-1, nkb), keep)
    # the same log-sum-exp, to rounding, as the dense call's own
    lse_dense = torch.empty_like(lse)
    sd.attn_dense(qd, kd, vd, lse_out=lse_dense)
    assert (lse - lse_dense).abs().max() < 1e-5


@pytest.mark.parametrize("B,Hq,Hkv,L,D,bq,bk,rho", [
    (1, 2, 2, 1024, 128, 128, 64, 0.25),   # 128-row work-groups, whole tiles
    (1, 4, 2, 1000, 128, 64, 64, 0.2),     # 16 tiles, the last one 40 keys; last query block 40 rows
    (1, 2, 1, 960, 128, 128, 64, 0.3),     # an odd number of tiles: the last column has no partner
    (2, 2, 2, 600, 64, 32, 32, 0.5),       # 32-key columns, last one 24 keys
    (1, 2, 2, 992, 128, 32, 32, 0.5),      # an odd number of 32-key blocks
    (1, 2, 2, 960, 64, 64, 128, 0.3),      # the last 128-key block is one tile
    (1, 2, 1, 1000, 128, 128, 128, 0.3),
    (1, 1, 1, 20, 128, 128, 32, 1.0),      # a single partial tile
    (1, 1, 1, 65, 64, 32, 64, 0.5),        # one key and one row in the last tile
    (3, 100, 100, 130, 64, 64, 64, 0.4),   # 256-row work-groups, more tiles than resident work-groups
    (2, 140, 70, 260, 128, 32, 128, 0.5),  # the same, two tiles a head, the second one 4 rows
])
def test_dense_select_bf16(B, Hq, Hkv, L, D, bq, bk, rho):
    _check(*_qkv(B, Hq, Hkv, L, D, torch.bfloat16, seed=L + bq + bk, scale=0.45 if D == 128 else 0.6), bq, bk, rho)


def test_dense_select_f32():
    _check(*_qkv(1, 2, 1, 200, 64, torch.float32, seed=3, scale=0.6), 32, 64, 0.4)


def test_dense_select_on_packed_views():
    g = torch.Generator().manual_seed(9)
    packed = (torch.randn(2, 333, 3, 3, 64, generator=g) * 0.6).to(torch.bfloat16)
    pd = packed.to(DEV)
    host = [packed[:, :, i].permute(0, 2, 1, 3) for i in range(3)]
    _check(*host, 64, 32, 0.3, views=[pd[:, :, i].permute(0, 2, 1, 3) for i in range(3)])


@pytest.mark.parametrize("bq,bk,L,D,H", [(128, 64, 1024, 128, 2), (64, 32, 600, 64, 2), (32, 128, 1000, 128, 2), (64, 64, 250, 64, 258)])
def test_dense_select_re_references_rows_whose_logits_climb(bq, bk, L, D, H):
    """Every row's logits climb by hundreds of octaves along the keys, so references are raised again and again and what
    a row has parked is rescaled each time. The pooled scores must match wherever the oracle's are representable."""
    g = torch.Generator().manual_seed(L + D)
    q = torch.zeros(1, H, L, D)
    k = torch.zeros(1, H, L, D)
    q[..., 0] = 8.0
    k[..., 0] = torch.linspace(0.0, 1.0, L) ** 2 * 40.0 * math.sqrt(D) / 8.0 * 8.0
    q[..., 1:] = 0.05 * torch.randn(1, H, L, D - 1, generator=g)
    k[..., 1:] = 0.05 * torch.randn(1, H, L, D - 1, generator=g)
    q, k = q.bfloat16(), k.bfloat16()
    v = torch.randn(1, H, L, D, generator=g).clamp(-2, 2).bfloat16()
    pooled = torch.empty(1, H, -(-L // bq), -(-L // bk), device=DEV)
    out, ix = sd.attn_dense_select(q.to(DEV), k.to(DEV), v.to(DEV), bq, bk, 0.3, pooled_out=pooled)
    sd.index_validate(ix)
    assert_output_close(out, oracle.attn_dense(q, k, v), torch.bfloat16, "dense+select climbing")
    _, _, apool, _ = oracle.select_pattern(q, k, bq, bk, 0.3)
    got = pooled.cpu().double().numpy()
    assert np.isfinite(got).all()
    # exponents of up to a few hundred octaves carry 2^-24 of their size: 600 octaves * ln 2 * 2^-24 = 2.5e-5
    big = apool > 1e-30
    assert (np.abs(got - apool)[big] / apool[big]).max() < 5e-5
    assert got[~big].max(initial=0.0) < 1e-29


def test_dense_select_per_sample_lengths():
    q, k, v = _qkv(3, 2, 2, 700, 128, torch.bfloat16, seed=5, scale=0.45)
    lens = [700, 333, 64]
    bq, bk, rho, nqb, nkb = 64, 64, 0.3, 11, 11
    out = torch.full(q.shape, 7.0, dtype=q.dtype, device=DEV)
    pooled = torch.zeros(3, 2, nqb, nkb, device=DEV)
    qd, kd, vd = (t.to(DEV) for t in (q, k, v))
    _, ix = sd.attn_dense_select(qd, kd, vd, bq, bk, rho, out=out, pooled_out=pooled,
                                 seq_lens=torch.tensor(lens, dtype=torch.int32, device=DEV))
    sd.index_validate(ix)
    for b, n in enumerate(lens):
        o1, ix1 = sd.attn_dense_select(qd[b:b + 1, :, :n], kd[b:b + 1, :, :n], vd[b:b + 1, :, :n], bq, bk, rho)
        assert torch.equal(out[b:b + 1, :, :n], o1) and (out[b, :, n:] == 7.0).all()
        used = ix1.row_ptr[0, 0, -1].item()
        assert torch.equal(ix.col_idx[b, :, :used], ix1.col_idx[0, :, :used])
        assert torch.equal(ix.row_ptr[b, :, :-(-n // bq) + 1], ix1.row_ptr[0])


def test_schedule_switch_step_equals_dense_then_select():
    q, k, v = _qkv(1, 4, 4, 1000, 128, torch.bfloat16, seed=8, scale=0.45)
    qd, kd, vd = (t.to(DEV) for t in (q, k, v))
    layer = sd.SparseDLayer(5, 0.2, 64, 64, 0.2)
    out = layer.step(qd, kd, vd, 0)
    assert layer.calls == {"dense": 1, "select": 1, "sparse": 0}
    assert_output_close(out, oracle.attn_dense(q, k, v), torch.bfloat16, "switch step")
    _, col_idx, apool, _ = oracle.select_pattern(q, k, 64, 64, 0.2)
    keep = oracle.kept_blocks(0.2, 16)
    compare_index(layer.index.col_idx.cpu().numpy(), col_idx, apool.reshape(-1, 16), keep)


@pytest.mark.parametrize("D,bq,bk", [(64, 64, 64), (128, 128, 128), (64, 32, 32), (128, 64, 128)])
@pytest.mark.parametrize("H,L", [(1, 700), (1, 1700), (60, 700)])   # one kernel of 128 rows a work-group; two kernels; 256 rows
@pytest.mark.parametrize("start", [-131, -145])
def test_parked_sums_far_above_a_reference_that_is_raised(start, H, L, D, bq, bk):
    """Keys far below the others, then some 55 octaves above those, then the others: the reference is raised by 130 octaves or more,
    and the sums parked so far by 2^55 relative to it still count."""
    octaves = torch.zeros(L)
    octaves[:64], octaves[64:192], octaves[192:320] = start, start + 50, start + 55
    q, k = torch.zeros(1, H, L, D), torch.zeros(1, H, L, D)
    q[..., 0] = 8
    k[0, :, :, 0] = octaves / 1.4426950408889634 * D ** 0.5 / 8
    q, k = q.bfloat16().to(DEV), k.bfloat16().to(DEV)
    nkb = -(-L // bk)
    p = torch.softmax(q[0, 0, :1].double() @ k[0, 0].double().t() / D ** 0.5, 1)[0]
    want = torch.stack([p[J * bk:(J + 1) * bk].mean() for J in range(nkb)])
    out = torch.zeros(1, H, -(-L // bq), nkb, device=DEV)
    sd.attn_dense_select(q, k, k, bq, bk, 0.5, pooled_out=out)
    held = want > 1e-34
    # arguments of up to 145 octaves, three roundings: 145 * 3 * 2^-24 * ln 2 = 1.8e-5
    assert held[256 // bk - 1] and ((out.double() - want).abs() / want)[..., held].max() < 3e-5
    assert (out[..., ~held] < 1e-33).all()
