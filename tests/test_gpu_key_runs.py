"""One-pass pooled scores with the keys in one run and in two: calls on both sides of the rule that chooses (units of 128 rows:
up to 256 of 24 key tiles or more, 30 at head dim 128, or a last round of 1024 that is at most half full if the units are long), and tile
counts at which the second run is shorter than the first. Scores against the pooling kernel that is given the row statistics."""
import pytest
import torch

import paper_2509_24014_amd as sd

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("B,H,L,D,bq,bk", [
    (1, 2, 1472, 64, 64, 64), (1, 2, 1473, 64, 128, 128),                # 23 and 24 tiles
    (1, 2, 1856, 128, 32, 32), (1, 1, 1857, 128, 64, 128), (1, 2, 2200, 128, 128, 64), (1, 2, 1728, 64, 32, 32),  # 29, 30, 35, 27 tiles
    (3, 2, 2300, 128, 32, 64), (4, 1, 1500, 64, 64, 128),                  # with lengths per sample: runs of 8, 7 and of 6, 4 tiles and so on
    (3, 4, 2200, 128, 128, 128), (2, 2, 1600, 64, 64, 32),                 # and of samples of 1 or 2 tiles (below)
    (1, 20, 1600, 64, 128, 64),                                            # 260 units: one run
    (1, 94, 2000, 64, 32, 128), (1, 87, 2300, 128, 128, 32), (1, 130, 1025, 64, 64, 64),  # 1504, 1566 and 1170 units
    (1, 165, 1000, 128, 64, 64), (1, 129, 1000, 128, 128, 64), (1, 240, 1020, 64, 64, 128),  # 1320 (two runs), 1032 and 1920 (one)
    (1, 342, 300, 64, 32, 128), (1, 769, 250, 64, 128, 64), (1, 770, 190, 128, 128, 64),  # 1026 and 1538 units of 3 to 5 tiles: one run
])
def test_scores_of_both_forms(B, H, L, D, bq, bk):
    g = torch.Generator(device=DEV).manual_seed(L)
    q = (torch.randn(B, H, L, D, generator=g, device=DEV) * 0.6).to(torch.bfloat16)
    k = (torch.randn(B, 1, L, D, generator=g, device=DEV) * 0.6).to(torch.bfloat16)
    nqb, nkb = -(-L // bq), -(-L // bk)
    lse, out = torch.zeros(B, H, L, dtype=torch.float32, device=DEV), torch.zeros(B, H, nqb, nkb, device=DEV)
    want = torch.zeros_like(out)
    for lens in (None, torch.tensor([L] + [max(1, L * 2 // 5)] * (B - 1), dtype=torch.int32, device=DEV),
                 torch.tensor([L, 64, 65, 130][:B], dtype=torch.int32, device=DEV)):   # runs of 1 and 0, 2 and 0, 2 and 1 tiles
        out.zero_()
        want.zero_()
        ix = sd.select_pattern(q, k, bq, bk, 0.3, pooled_out=out, seq_lens=lens)
        sd.index_validate(ix)
        sd.attn_dense(q, k, k, seq_lens=lens, lse_out=lse)
        sd.select_pattern(q, k, bq, bk, 0.3, pooled_out=want, lse_in=lse, seq_lens=lens)
        # each is within 5e-6 of the exact score (the bar of the pooling kernels)
        for b in range(B):
            n = L if lens is None else int(lens[b])
            x, y = out[b, :, :-(-n // bq), :-(-n // bk)], want[b, :, :-(-n // bq), :-(-n // bk)]
            assert torch.isfinite(x).all() and ((x - y).abs() <= 1e-5 * y).all(), ((x - y).abs() / y).max()


@pytest.mark.parametrize("D,where", [(64, 100), (64, 1500), (128, 40), (128, 1000), (128, 2299)])
def test_a_logit_far_above_the_others_in_either_run(D, where):
    """One key whose logits are 150 to 300 octaves above every other key's: the references of the runs differ by as much, and
    all of the weight is in one column."""
    L, b = 2304, 64
    q = torch.ones(1, 1, L, D, device=DEV, dtype=torch.bfloat16)
    q[:, :, 1152:] = 2
    k = torch.full((1, 1, L, D), -0.25, device=DEV, dtype=torch.bfloat16)
    k[:, :, where] = 104 * D ** -0.5   # logits (104 + sqrt(D) / 4) times 1 and 2 above the others
    out = torch.zeros(1, 1, L // b, L // b, device=DEV)
    sd.select_pattern(q, k, b, b, 0.3, pooled_out=out)
    want = torch.zeros_like(out)
    want[..., where // b] = 1 / b
    assert torch.allclose(out, want, rtol=5e-6, atol=1e-30)


@pytest.mark.parametrize("D,bq,bk", [(64, 64, 64), (128, 128, 128), (64, 32, 32), (128, 64, 128)])
@pytest.mark.parametrize("run,low,high", [(0, -130, -35), (1, -130, -35), (1, -180, -90), (0, -180, -90), (1, -250, -155)])
def test_scores_of_a_run_whose_reference_is_far_below(run, low, high, D, bq, bk):
    """One run begins 130 octaves or more below the other, its reference with it, and climbs by 90 to 95, too little for the
    reference to be raised: the factor between the references is below the smallest float, the scores are not. Also the two
    parts of a boundary block among the keys that climb."""
    L = 2305 if bk < 128 else 2304 + 65   # 37 or 38 tiles, the first run 20 of them, keys 0 .. 1279
    octaves = torch.zeros(L)
    begin = 1280 * run
    octaves[begin:L if run else 1280] = low
    octaves[begin + 400:begin + 600] = high
    q, k = torch.zeros(1, 2, L, D), torch.zeros(1, 2, L, D)
    q[..., 0] = 8
    k[0, :, :, 0] = octaves / 1.4426950408889634 * D ** 0.5 / 8
    q, k = q.bfloat16().to(DEV), k.bfloat16().to(DEV)
    nqb, nkb = -(-L // bq), -(-L // bk)
    p = torch.softmax(q[0, 0, :1].double() @ k[0, 0].double().t() / D ** 0.5, 1)[0]
    want = torch.stack([p[J * bk:(J + 1) * bk].mean() for J in range(nkb)])
    out = torch.zeros(1, 2, nqb, nkb, device=DEV)
    ix = sd.select_pattern(q, k, bq, bk, 0.5, pooled_out=out)
    # arguments of up to 250 octaves are carried to 2^-24 of that, at three roundings: 250 * 3 * 2^-24 * ln 2 = 3.1e-5
    held = want > 1e-34
    assert held.sum() >= nkb // 2 and ((out.double() - want).abs() / want)[..., held].max() < 4e-5
    assert (out[..., ~held] < 1e-33).all()
    keep = sd.kept_blocks(0.5, nkb)
    cut = want.sort(descending=True).values[keep - 1]
    if cut > 1e-34:
        assert (want[ix.col_idx.view(1, 2, nqb, keep).long()] >= cut * (1 - 1e-4)).all()
    token = begin + 500 + 5   # inside a key block, among the keys that climb
    js = token // bk
    parts = [p[js * bk:token].mean(), p[token:(js + 1) * bk].mean()]
    ix = sd.select_pattern_isolated_tokens(q, k, bq, bk, 0.5, token)
    sd.index_validate(ix)
    first = torch.cat([want[:js], parts[0][None]])
    kept = sd.kept_blocks(0.5, js + 1)
    rows = ix.row_ptr[0, 0].tolist()
    for I in range(nqb):
        row = ix.col_idx[0, 0, rows[I]:rows[I + 1]].tolist()
        mine = [j for j in row if j < js]
        floor = first.sort(descending=True).values[kept - 1]
        assert all(want[j] >= floor * (1 - 1e-4) for j in mine)


@pytest.mark.parametrize("D,bq,bk", [(64, 64, 64), (128, 128, 128), (64, 32, 32)])
@pytest.mark.parametrize("L", [700, 2300])   # one run of keys, two
@pytest.mark.parametrize("start", [-130, -150, -185])
def test_parked_sums_far_above_a_reference_that_is_raised(start, L, D, bq, bk):
    """Within one run: keys far below the others, then some 95 octaves above those, then the others: the reference is raised by 130
    octaves or more, and the sums parked so far by 2^95 relative to it still count."""
    octaves = torch.zeros(L)
    octaves[:64], octaves[64:192], octaves[192:320] = start, start + 90, start + 95
    q, k = torch.zeros(1, 1, L, D), torch.zeros(1, 1, L, D)
    q[..., 0] = 8
    k[0, 0, :, 0] = octaves / 1.4426950408889634 * D ** 0.5 / 8
    q, k = q.bfloat16().to(DEV), k.bfloat16().to(DEV)
    nkb = -(-L // bk)
    p = torch.softmax(q[0, 0, :1].double() @ k[0, 0].double().t() / D ** 0.5, 1)[0]
    want = torch.stack([p[J * bk:(J + 1) * bk].mean() for J in range(nkb)])
    out = torch.zeros(1, 1, -(-L // bq), nkb, device=DEV)
    sd.select_pattern(q, k, bq, bk, 0.5, pooled_out=out)
    held = want > 1e-34
    # arguments of up to 185 octaves, three roundings: 185 * 3 * 2^-24 * ln 2 = 2.3e-5
    assert held[64 // bk + (bk == 128)] and ((out.double() - want).abs() / want)[..., held].max() < 3e-5
    assert (out[..., ~held] < 1e-33).all()


@pytest.mark.parametrize("bk", [32, 64, 128])
@pytest.mark.parametrize("n", [1, 40, 64, 65, 100, 130])
def test_a_sample_of_a_tile_or_two_beside_a_long_one(n, bk):
    """The long sample takes two runs; the first run of a sample of one tile is that tile, half a block of 128."""
    g = torch.Generator(device=DEV).manual_seed(n)
    q, k = ((torch.randn(2, 2, 2300, 64, generator=g, device=DEV) * 0.6).to(torch.bfloat16) for _ in range(2))
    out = torch.full((2, 2, 36, -(-2300 // bk)), 7.0, device=DEV)
    sd.select_pattern(q, k, 64, bk, 0.3, pooled_out=out, seq_lens=torch.tensor([2300, n], dtype=torch.int32, device=DEV))
    p = torch.softmax(q[1, :, :n].double() @ k[1, :, :n].double().transpose(1, 2).contiguous() / 8, 2)
    for I in range(-(-n // 64)):
        for J in range(-(-n // bk)):
            want = p[:, I * 64:(I + 1) * 64, J * bk:(J + 1) * bk].mean((1, 2))
            assert ((out[1, :, I, J].double() - want).abs() <= 5e-6 * want).all(), (I, J)
    assert (out[1, :, -(-n // 64):] == 7.0).all() and (out[1, :, :, -(-n // bk):] == 7.0).all()
