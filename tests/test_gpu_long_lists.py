"""Lists of more than 64 tiles: a wave keeps the block numbers of 64 steps of its tile stream in a register and fetches the next
ones on the way. Every form of the split-key kernel, around the lengths at which it does."""
import math

import pytest
import torch

import paper_2509_24014_amd as sd

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("bq,bk,H", [
    (64, 64, 1), (64, 64, 6),      # two streams; up to 512 runs of 32 rows: 2 x 4 parts
    (64, 64, 10), (64, 128, 10),   # one stream, two row groups
    (32, 32, 1), (32, 64, 10),     # two streams without barriers; one
])
def test_lists_around_the_register_length(bq, bk, H, D):
    L = 2 * 64 * 67 - 17     # 134 tiles, the last one partial
    nqb, nkb = -(-L // bq), -(-L // bk)
    g = torch.Generator(device=DEV).manual_seed(bq + bk + H)
    q, k, v = [torch.randn(1, H, L, D, generator=g, device=DEV).bfloat16() for _ in range(3)]
    unit = 64 / bk           # listed blocks a tile
    lengths = [int(round(t * unit)) for t in (0, 1, 59, 60, 61, 62, 63, 64, 65, 66, 121, 123, 124, 125, 126, 127, 128, 129, 130, 133)]
    row, cols, masks = [0], [], {}
    for i in range(nqb):
        n = min(lengths[i % len(lengths)], nkb)
        c = torch.randperm(nkb, generator=g, device=DEV)[:n].sort().values
        if n and i % 2:
            c[-1] = nkb - 1  # ascending still, and the partial block listed (unless it was already)
        cols.append(c)
        row.append(row[-1] + n)
    col = torch.cat(cols).to(torch.int32)
    ix = sd.BlockIndex(torch.tensor(row, dtype=torch.int32, device=DEV).expand(1, H, nqb + 1).contiguous(),
                       col.expand(1, H, len(col)).contiguous(), bq, bk, nkb)
    sd.index_validate(ix)
    out = sd.attn_sparse(q, k, v, ix)
    for h in (0, H - 1):
        for i in list(range(0, len(lengths))) + [nqb - 1]:
            r = slice(i * bq, min((i + 1) * bq, L))
            keys = (cols[i][:, None] * bk + torch.arange(bk, device=DEV)).flatten()
            keys = keys[keys < L]
            if len(keys) == 0:
                assert not out[0, h, r].any()
                continue
            s = q[0, h, r].double() @ k[0, h, keys].double().t() / math.sqrt(D)
            d = (out[0, h, r].double() - torch.softmax(s, 1) @ v[0, h, keys].double()).abs()
            assert d.max() < 2e-2 and d.mean() < 2e-3, (h, i, len(keys), d.max())
