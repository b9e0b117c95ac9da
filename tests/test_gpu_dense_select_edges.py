"""The switch step in one call at its edges: a missing or short workspace, a stream that is not the current one, and replays
from a HIP graph."""
import pytest
import torch

import paper_2509_24014_amd as sd

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
WORKSPACE = 7   # SPARSED_ERR_WORKSPACE


def _inputs(dtype, B=1, H=2, L=700, D=64, seed=1):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return [(torch.randn(B, H, L, D, device=DEV, generator=g) * s).to(dtype) for s in (0.6, 0.6, 1.0)]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_a_workspace_that_is_too_small_or_misaligned_is_refused_before_anything_runs(dtype):
    q, k, v = _inputs(dtype)
    bq, bk, rho = 64, 32, 0.3
    # the exact need: pooled scores and one slab column set per work-group (bf16), statistics and pooled scores (fp32)
    need = next(n for n in range(256, sd.select_workspace_bytes(q, bq, bk) + 1, 256) if _accepts(q, k, v, bq, bk, rho, n))
    for n in (0, need - 256):
        out = torch.full_like(q, 7.0)
        with pytest.raises(sd.SparsedError) as e:
            sd.attn_dense_select(q, k, v, bq, bk, rho, out=out, workspace=torch.empty(n, dtype=torch.uint8, device=DEV))
        assert e.value.status == WORKSPACE
        assert (out == 7.0).all()
    with pytest.raises(sd.SparsedError) as e:
        sd.attn_dense_select(q, k, v, bq, bk, rho, workspace=torch.empty(need + 512, dtype=torch.uint8, device=DEV)[16:])
    assert e.value.status == WORKSPACE
    # and with exactly the need, guarded on both sides, nothing outside it is written
    buf = torch.full((need + 512,), 0xA5, dtype=torch.uint8, device=DEV)
    out, ix = sd.attn_dense_select(q, k, v, bq, bk, rho, workspace=buf[256:256 + need])
    want, want_ix = sd.attn_dense_select(q, k, v, bq, bk, rho)
    assert (buf[:256] == 0xA5).all() and (buf[256 + need:] == 0xA5).all()
    assert torch.equal(out, want) and torch.equal(ix.col_idx, want_ix.col_idx) and torch.equal(ix.row_ptr, want_ix.row_ptr)


def _accepts(q, k, v, bq, bk, rho, n):
    try:
        sd.attn_dense_select(q, k, v, bq, bk, rho, workspace=torch.empty(n, dtype=torch.uint8, device=DEV))
        return True
    except sd.SparsedError as e:
        assert e.status == WORKSPACE
        return False


def test_on_another_stream_everything_the_call_allocates_is_kept_for_it(monkeypatch):
    q, k, v = _inputs(torch.bfloat16)
    want, want_ix = sd.attn_dense_select(q, k, v, 64, 64, 0.3)
    recorded = []
    real = torch.Tensor.record_stream
    monkeypatch.setattr(torch.Tensor, "record_stream", lambda t, s: (recorded.append((t.data_ptr(), s)), real(t, s))[1])
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    out, ix = sd.attn_dense_select(q, k, v, 64, 64, 0.3, stream=side)
    side.synchronize()
    assert torch.equal(out, want) and torch.equal(ix.col_idx, want_ix.col_idx)
    for t in (out, ix.row_ptr, ix.col_idx):
        assert (t.data_ptr(), side) in recorded
    assert len(recorded) == 4   # and the workspace
    recorded.clear()
    sd.attn_dense_select(q, k, v, 64, 64, 0.3)
    assert not recorded


def test_replays_from_a_hip_graph():
    """Replays on new contents of the same buffers, with eager work and synchronisation between them, equal the eager call bit
    for bit every time; the schedule's own step is captured the same way."""
    B, H, L, D, bq, bk, rho = 1, 4, 1000, 128, 64, 64, 0.25
    q, k, v = _inputs(torch.bfloat16, B, H, L, D)
    out, nqb, nkb = torch.empty_like(q), -(-L // bq), -(-L // bk)
    index = sd.BlockIndex(torch.empty(B, H, nqb + 1, dtype=torch.int32, device=DEV),
                          torch.empty(B, H, nqb * sd.kept_blocks(rho, nkb), dtype=torch.int32, device=DEV), bq, bk, nkb)
    pooled = torch.empty(B, H, nqb, nkb, device=DEV)
    ws = torch.empty(sd.select_workspace_bytes(q, bq, bk), dtype=torch.uint8, device=DEV)
    layer, out_layer = sd.SparseDLayer(5, 0.2, bq, bk, rho), torch.empty_like(q)

    def step():
        sd.attn_dense_select(q, k, v, bq, bk, rho, out=out, workspace=ws, pooled_out=pooled, index=index)
        layer.step(q, k, v, 0, out=out_layer)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for trial in range(4):
        for t in (q, k, v):
            t.copy_(torch.randn(B, H, L, D, device=DEV).to(torch.bfloat16))
        for t in (out, out_layer, pooled):
            t.fill_(float("nan"))
        index.col_idx.fill_(-1)
        layer.index.col_idx.fill_(-1)
        graph.replay()
        torch.cuda.synchronize()
        pooled_e = torch.empty_like(pooled)
        out_e, index_e = sd.attn_dense_select(q, k, v, bq, bk, rho, pooled_out=pooled_e)
        assert torch.equal(out, out_e) and torch.equal(out_layer, out_e) and torch.equal(pooled, pooled_e), f"replay {trial}"
        for ix in (index, layer.index):
            assert torch.equal(ix.col_idx, index_e.col_idx) and torch.equal(ix.row_ptr, index_e.row_ptr), f"replay {trial}: index"


@pytest.mark.parametrize("H,L,D,bq,bk", [(100, 300, 64, 64, 64), (90, 270, 128, 32, 128), (130, 390, 64, 128, 32)])
def test_padded_batches_over_many_units_equal_single_samples(H, L, D, bq, bk):
    """More row tiles than resident work-groups, of which whole runs do not exist in the shorter samples: every persistent
    work-group steps over some and reuses its slab after others. Both kernels that park block sums."""
    rho, lens = 0.3, [L, L // 3, 0, L // 2 + 1]
    q, k, v = _inputs(torch.bfloat16, len(lens), H, L, D)
    sl = torch.tensor(lens, dtype=torch.int32, device=DEV)
    nqb, nkb = -(-L // bq), -(-L // bk)
    one, own = (torch.full((len(lens), H, nqb, nkb), -1.0, device=DEV) for _ in range(2))
    out = torch.full_like(q, 7.0)
    _, ix = sd.attn_dense_select(q, k, v, bq, bk, rho, out=out, pooled_out=one, seq_lens=sl)
    ix_own = sd.select_pattern(q, k, bq, bk, rho, pooled_out=own, seq_lens=sl)
    for b, n in enumerate(lens):
        assert (out[b, :, n:] == 7.0).all()
        if n == 0:
            assert (one[b] == -1.0).all() and (own[b] == -1.0).all()
            assert not ix.row_ptr[b].any() and not ix_own.row_ptr[b].any()
            continue
        q1, k1, v1 = (t[b:b + 1, :, :n] for t in (q, k, v))
        nq, nk = -(-n // bq), -(-n // bk)
        p1 = torch.full((1, H, nq, nk), -1.0, device=DEV)
        o1, ix1 = sd.attn_dense_select(q1, k1, v1, bq, bk, rho, pooled_out=p1)
        assert torch.equal(out[b:b + 1, :, :n], o1)   # a row does not depend on its work-group
        used = ix1.row_ptr[0, 0, -1].item()
        for pooled, index in ((one, ix), (own, ix_own)):
            torch.testing.assert_close(pooled[b:b + 1, :, :nq, :nk], p1, rtol=5e-6, atol=0)
            assert (pooled[b, :, nq:] == -1.0).all() and (pooled[b, :, :, nk:] == -1.0).all()
            assert torch.equal(index.row_ptr[b, :, :nq + 1], ix1.row_ptr[0])
        assert torch.equal(ix.col_idx[b, :, :used], ix1.col_idx[0, :, :used])
