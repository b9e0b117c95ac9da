"""Timed cases of the attention path: what a program that runs SparseD on one layer calls, from the smallest call to
the longest context.

A case is a plain dict. ``kind`` says which calls a pass makes, through the public entry points:

  dense     one full-attention step (``attn_dense``)
  sparse    one reuse step with a stored pattern (``attn_sparse``)
  switch    the last dense step of a schedule, which also selects the pattern (``SparseDLayer.step``)
  select    a selection without a dense call at the same step, scores kept beside the index (``select_pattern``)
  isolated  a padded batch of samples of different length: selection with the prefill boundary at a token
            (``select_pattern_isolated_tokens``) and the sparse step on it
  schedule  a whole short schedule with drifting inputs: dense steps, the switch, sparse steps (``SparseDLayer.step``)

Shapes and block settings are those of ``workload/configs.py`` and of the tests; the other lengths are generic.
"""
import math

import torch

import paper_2509_24014_amd as sd
import workload

DEVICE = "cuda"


def listed():
    bf16, f32 = "bf16", "f32"
    return [
        # the tiny fp32 schedule, whole (1 dense step with selection, 4 sparse steps): the latency of small calls
        _case("tiny_schedule_f32", "schedule", f32, 1, 2, 2, 256, 64, 32, 32, 0.3, steps=5),
        # a short ragged dense step, grouped heads, head dim 64, two samples: a call that cannot fill the chip
        _case("dense_600_gqa_d64", "dense", bf16, 2, 8, 2, 600, 64),
        # dense step at 4k
        _case("dense_4k", "dense", bf16, 1, 32, 32, 4096, 128),
        # dense step of a grouped-query layer (28 query heads over 4) at 32k
        _case("dense_32k_gqa", "dense", bf16, 1, 28, 4, 32768, 128),
        # reuse step with the short-context setting (32 x 32 blocks, half of them kept), length not a block multiple
        _case("sparse_2000_32x32", "sparse", bf16, 1, 32, 32, 2000, 128, 32, 32, 0.5),
        # reuse step at 4k: where a denoising loop spends most of its calls
        _case("sparse_4k", "sparse", bf16, 1, 32, 32, 4096, 128, 64, 64, 0.2),
        # reuse step at the long context
        _case("sparse_64k", "sparse", bf16, 1, 32, 32, 65536, 128, 128, 64, 0.05),
        # dense step + selection at 4k
        _case("switch_4k", "switch", bf16, 1, 32, 32, 4096, 128, 64, 64, 0.2),
        # dense step + selection at the long context: the largest pass
        _case("switch_64k", "switch", bf16, 1, 32, 32, 65536, 128, 128, 64, 0.05),
        # selection without a dense call at the same step (selecting anew at a sparse step)
        _case("select_16k", "select", bf16, 1, 32, 32, 16384, 128, 64, 64, 0.1),
        # padded batch, prefill boundary inside a key block, head dim 64, long-context block setting
        _case("isolated_batch_3000_d64", "isolated", bf16, 3, 8, 8, 3000, 64, 128, 128, 0.3),
        # fp32 inputs at an ordinary size: dense + selection, then two sparse steps
        _case("schedule_2000_f32", "schedule", f32, 1, 8, 8, 2000, 128, 64, 64, 0.2, steps=3),
    ]


def _case(name, kind, dtype, B, Hq, Hkv, L, D, bq=0, bk=0, rho=0.0, steps=0):
    c = dict(kind=kind, dtype=dtype, B=B, Hq=Hq, Hkv=Hkv, L=L, D=D)
    if bq:
        c.update(bq=bq, bk=bk, rho=rho)
    if steps:
        c["steps"] = steps
    return dict(name=name, **c) if name else c


def draw(rng):
    """One more case: kind, heads, block setting and (log-uniform, mostly ragged) length drawn over the same ranges."""
    kind = rng.choice(["dense", "dense", "sparse", "sparse", "switch", "switch", "select", "isolated", "schedule"])
    D = rng.choice([64, 128, 128])
    B, Hq, Hkv = rng.choice([(1, 4, 4), (1, 8, 2), (2, 8, 8), (1, 28, 4), (1, 32, 32)])
    # (block_q, block_k, rho): the named workloads' settings, the paper's two square ones, and one between them
    bq, bk, rho = rng.choice([(32, 32, 0.5), (64, 64, 0.2), (64, 64, 0.1), (128, 64, 0.1), (128, 64, 0.05), (128, 128, 0.3)])
    lo, hi = 256, 32768
    if kind == "schedule":                       # fp32: up to a few thousand tokens
        Hq, Hkv, hi = min(Hq, 8), min(Hkv, 8), 3000
        if Hq % Hkv:
            Hkv = 2
    elif kind == "isolated":
        B, Hq, Hkv, lo, hi = rng.choice([2, 3, 4]), rng.choice([4, 8, 16]), 0, 512, 8192
        Hkv = Hq // rng.choice([1, 2])
    L = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.4:
        L = max(lo, L // 256 * 256)
    if kind == "dense":
        return _case("", kind, "bf16", B, Hq, Hkv, L, D)
    if kind == "schedule":
        return _case("", kind, "f32", B, Hq, Hkv, L, D, bq, bk, rho, steps=rng.choice([3, 4, 5]))
    return _case("", kind, "bf16", B, Hq, Hkv, L, D, bq, bk, rho)


# ------------------------------------------------------------------------------------------------ inputs


def _lengths(case):
    """Per-sample lengths of a padded batch: the first sample is full, the others get shorter."""
    return [max(1, case["L"] * (10 - 3 * b) // 10) for b in range(case["B"])]


def _prefill(case):
    """A prefill boundary that lies inside a key block whenever blocks have more than one token."""
    p = case["L"] * 6 // 10
    return p + 1 if p % case["bk"] == 0 else p


def _inputs(case, seed):
    cfg = workload.get_config("llada4k").scaled(
        name=case["kind"], B=case["B"], Hq=case["Hq"], Hkv=case["Hkv"], L=case["L"], d=case["D"], dtype=case["dtype"],
        sigma=0.02 if case["kind"] == "schedule" else 0.0,
        # head-specific structure needs 128 features; plain normal Q, K, V there and where attention runs on a pattern
        # selected in the same pass (planted heads without structure have near-ties in most rows, and a tie that falls
        # the other way would be another, equally good, attention output)
        planted=case["D"] >= 128 and case["kind"] not in ("isolated", "schedule"))
    return workload.make_inputs(cfg, seed=seed, device=DEVICE)


def _block_means(x, block):
    """[B, H, L, D] -> [B, H, ceil(L / block), D], the last block over the rows that exist."""
    B, H, L, D = x.shape
    n = -(-L // block)
    pad = torch.zeros(B, H, n * block - L, D, dtype=x.dtype, device=x.device)
    total = torch.cat([x, pad], dim=2).view(B, H, n, block, D).sum(3)
    rows = torch.full((n,), block, device=x.device)
    rows[-1] = L - (n - 1) * block
    return total / rows.view(1, 1, n, 1)


def _stored_index(case, q, k):
    """A stored pattern for the reuse step: per head and query block the key blocks whose mean key answers the mean
    query most (the same structure as a selected pattern: windows, stripes, segments, scattered blocks)."""
    B, Hq, L = case["B"], case["Hq"], case["L"]
    qm, km = _block_means(q.float(), case["bq"]), _block_means(k.float(), case["bk"])
    km = km.repeat_interleave(Hq // case["Hkv"], dim=1)
    score = torch.matmul(qm, km.transpose(2, 3).contiguous())
    nqb, nkb = score.shape[2], score.shape[3]
    keep = sd.kept_blocks(case["rho"], nkb)
    col = score.topk(keep, dim=3).indices.sort(dim=3).values.to(torch.int32).reshape(B, Hq, nqb * keep).contiguous()
    row = (torch.arange(nqb + 1, device=q.device, dtype=torch.int32) * keep).expand(B, Hq, nqb + 1).contiguous()
    return sd.BlockIndex(row, col, case["bq"], case["bk"], nkb)


def _empty_index(case, keep):
    """Buffers of an index to be selected, zeroed: shorter samples leave the end of theirs unwritten."""
    B, Hq, nqb, nkb = case["B"], case["Hq"], -(-case["L"] // case["bq"]), -(-case["L"] // case["bk"])
    return sd.BlockIndex(torch.zeros(B, Hq, nqb + 1, dtype=torch.int32, device=DEVICE),
                         torch.zeros(B, Hq, max(nqb * keep, 1), dtype=torch.int32, device=DEVICE), case["bq"], case["bk"], nkb)


def prepare(case, seed):
    kind = case["kind"]
    inp = _inputs(case, seed)
    q, k, v = inp.rounded()
    s = dict(kind=kind, q=q, k=k, v=v)
    if kind not in ("select", "schedule"):
        s["out"] = torch.zeros_like(q)
    if kind == "sparse":
        s["index"] = _stored_index(case, q, k)
    elif kind == "switch":
        s["layer"] = sd.SparseDLayer(5, 0.2, case["bq"], case["bk"], case["rho"])   # step 0 is the last dense step
    elif kind == "select":
        bq, bk, nkb = case["bq"], case["bk"], -(-case["L"] // case["bk"])
        s.update(index=_empty_index(case, sd.kept_blocks(case["rho"], nkb)), rho=case["rho"], bq=bq, bk=bk,
                 workspace=torch.empty(sd.select_workspace_bytes(q, bq, bk), dtype=torch.uint8, device=DEVICE),
                 pooled=torch.zeros(case["B"], case["Hq"], -(-case["L"] // bq), nkb, dtype=torch.float32, device=DEVICE))
    elif kind == "isolated":
        p, bk, nkb = _prefill(case), case["bk"], -(-case["L"] // case["bk"])
        keep = sd.kept_blocks(case["rho"], -(-p // bk)) + sd.kept_blocks(case["rho"], nkb - p // bk)
        s.update(index=_empty_index(case, keep), prefill=p, rho=case["rho"], bq=case["bq"], bk=bk,
                 seq_lens=torch.tensor(_lengths(case), dtype=torch.int32, device=DEVICE))
    elif kind == "schedule":
        s["layer"] = sd.SparseDLayer(case["steps"], 0.2, case["bq"], case["bk"], case["rho"])
        s["qkv"] = []
        for t in range(case["steps"]):
            if t:
                inp.advance()
            s["qkv"].append(tuple(x.clone() for x in inp.rounded()))   # fp32: rounded() is the drifting master itself
    return s


def run(s):
    kind, q, k, v = s["kind"], s["q"], s["k"], s["v"]
    if kind == "dense":
        return sd.attn_dense(q, k, v, out=s["out"])
    if kind == "sparse":
        return sd.attn_sparse(q, k, v, s["index"], out=s["out"])
    if kind == "select":
        ix = sd.select_pattern(q, k, s["bq"], s["bk"], s["rho"], workspace=s["workspace"], pooled_out=s["pooled"], index=s["index"])
        return s["pooled"], ix.row_ptr, ix.col_idx
    if kind == "isolated":
        ix = sd.select_pattern_isolated_tokens(q, k, s["bq"], s["bk"], s["rho"], s["prefill"], index=s["index"], seq_lens=s["seq_lens"])
        out = sd.attn_sparse(q, k, v, ix, out=s["out"], seq_lens=s["seq_lens"])
        return out, ix.row_ptr, ix.col_idx
    layer = s["layer"]
    if kind == "schedule":
        outs = [layer.step(qt, kt, vt, t) for t, (qt, kt, vt) in enumerate(s["qkv"])]
        return outs, layer.index.row_ptr, layer.index.col_idx
    out = layer.step(q, k, v, 0, out=s["out"])   # switch
    return out, layer.index.row_ptr, layer.index.col_idx


# ------------------------------------------------------------------------------------------------ accounting


def work(case):
    """Inputs read once, outputs written once; matrix products of the attended pairs, S = Q K^T once per step."""
    el = 2 if case["dtype"] == "bf16" else 4
    kind, B, Hq, Hkv, L, D = case["kind"], case["B"], case["Hq"], case["Hkv"], case["L"], case["D"]
    lens = _lengths(case) if kind == "isolated" else [L] * B
    tokens, pairs = sum(lens), sum(n * n for n in lens)
    step_bytes = tokens * D * el * (2 * Hq + 2 * Hkv)
    dense = 4.0 * Hq * pairs * D
    if kind == "dense":
        return {"bytes": step_bytes, "flops": dense}
    nqb, nkb = -(-L // case["bq"]), -(-L // case["bk"])
    keep = sd.kept_blocks(case["rho"], nkb)
    index = 4 * B * Hq * nqb * keep
    sparse = dense * min(1.0, keep * case["bk"] / L)
    if kind == "sparse":
        return {"bytes": step_bytes + index, "flops": sparse}
    if kind == "switch":
        return {"bytes": step_bytes + index, "flops": dense}
    if kind == "select":
        return {"bytes": tokens * D * el * (Hq + Hkv) + index + 4 * B * Hq * nqb * nkb, "flops": dense / 2}
    if kind == "isolated":
        return {"bytes": step_bytes + index, "flops": dense / 2 + sparse}
    steps = case["steps"]
    return {"bytes": steps * step_bytes + index, "flops": dense + (steps - 1) * sparse}


def tolerance(case):
    """About four times what the path was seen to be off by: attention against float64 (bf16 2.4e-3, largest 1.6e-2;
    fp32 4e-7 to 1.6e-6), selection against itself with its sums in another order (scores as fp32 sums; 1e-4 to 5e-3 of
    the index entries: near-ties)."""
    if case["kind"] == "isolated":   # a tie that falls the other way changes that query block's attention
        return {"rel": 2e-2, "max": 0.9, "differ": 0.01}
    if case["dtype"] == "f32" or case["kind"] == "select":
        return {"rel": 1e-5, "max": 5e-5, "differ": 0.01}
    return {"rel": 1e-2, "max": 7e-2, "differ": 0.01}
