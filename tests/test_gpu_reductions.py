"""The two reduction kernels: what dropped columns cost them, and their rows written in bursts."""
import numpy as np
import pytest
import torch

import paper_2508_18224_amd as nsa
import workloads as wl

pytestmark = pytest.mark.gpu


def _reduction_times(seqlens, topk):
    """(fwd_merge, bwd_dq_reduce) in ms, the fastest of several, and the kept columns per row."""
    hkv, tokens = 16, sum(seqlens)
    w = wl.realise(wl.Workload("reductions", seqlens, hq=hkv, hkv=hkv, topk=topk, sink=True, seed=12), tensors=False)
    gen = torch.Generator(device="cuda").manual_seed(3)
    q, k, v, do = (torch.randn(tokens, hkv, 128, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(4))
    idx, cu = torch.from_numpy(w.idx).cuda(), torch.from_numpy(w.cu_seqlens).cuda()
    attn = nsa.SelAttention(tokens, hkv, hkv, topk, nseq=len(seqlens), dense=False)
    best = [float("inf")] * 2
    for _ in range(6):
        nsa.binding.profile_enable(64)
        o, lse = attn.forward(q, k, v, idx, cu)
        attn.backward(q, k, v, o, lse, do, cu)
        torch.cuda.synchronize()
        got = nsa.binding.profile_collect()
        best = [min(b, got[nm][0]) for b, nm in zip(best, ("fwd_merge", "bwd_dq_reduce"))]
    nsa.binding.profile_enable(0)
    return best, float((w.idx >= 0).mean()) * topk


@pytest.mark.parametrize("sequences", [24, 100])  # below and above the rows from which long sequences are written in bursts
def test_dropped_columns_are_not_gathered(sequences):
    """Rows of short sequences keep few of their columns: the reductions take the time of the rows they read and write, here about
    a sixth of what rows with all 32 columns take, not that of the columns there could be (which took half of it, three times the
    rows' share; now 1.2 to 1.4 times)."""
    print("case dropped columns", sequences, flush=True)
    lengths = np.random.default_rng(8).exponential(300, sequences).astype(int) + 1
    short, kept = _reduction_times([int(n) for n in lengths], 32)
    full, kept_full = _reduction_times([int(lengths.sum())], 32)
    rows = (kept + 1) / (kept_full + 1)
    print("share of rows", rows, "of the time", short[0] / full[0], short[1] / full[1], flush=True)
    assert rows < 0.25
    for a, b in zip(short, full):
        assert a < 2 * rows * b


@pytest.mark.parametrize("seqlens,heads,topk", [
    ([8200], 16, 9),             # dQ in bursts, two turns of the chip, workgroups of four and five steps; merged row by row
    ([16399], 32, 6),            # dQ in bursts, full workgroups
    ([16399], 16, 16),           # both: three turns, five and six steps, the last one part empty
    ([4000, 1, 12500], 32, 16),  # five turns of full workgroups; gated in bursts too
])
def test_bursts_of_rows_with_holes_match_row_by_row(seqlens, heads, topk):
    """Columns dropped anywhere in a row, rows that keep none, whole tokens that keep none: one pass writes in bursts, a KV head per
    pass row by row.  Same sums in the same order, same bits."""
    print("case holes", seqlens, heads, topk, flush=True)
    w = wl.realise(wl.Workload("holes", seqlens, hq=heads, hkv=heads, topk=topk, sink=True, seed=98), tensors=False)
    rng = np.random.default_rng(9)
    tokens = w.total_tokens
    w.idx[rng.random(w.idx.shape) < 0.3] = -1
    w.idx[rng.random(w.idx.shape[:2]) < 0.05] = -1
    w.idx[rng.integers(0, tokens, 300)] = -1
    w.idx[..., topk // 2] = w.idx[..., 0]
    gen = torch.Generator(device="cuda").manual_seed(5)
    q, k, v, do, acc = (torch.randn(tokens, heads, 128, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(5))
    gate = torch.rand(tokens, heads, generator=gen, device="cuda")
    idx, cu = torch.from_numpy(w.idx).cuda(), torch.from_numpy(w.cu_seqlens).cuda()
    outs = []
    for cap in (None, 1):
        attn = nsa.SelAttention(tokens, heads, heads, topk, nseq=len(seqlens), ws_cap_bytes=cap, dense=False)
        for ws in (attn.fwd_ws, attn.bwd_ws):
            ws.fill_(0x7F)
        o, lse = attn.forward(q, k, v, idx, cu)
        got = [o, lse, *attn.backward(q, k, v, o, lse, do, cu), *attn.forward_gated(q, k, v, idx, gate, acc, cu)]
        outs.append([x.clone() for x in got])
    for nm, a, b in zip(("O", "LSE", "dQ", "dK", "dV", "gated O_out", "gated O", "gated LSE"), *outs):
        assert torch.equal(a.view(torch.int16 if a.dtype == torch.bfloat16 else torch.int32),
                           b.view(torch.int16 if b.dtype == torch.bfloat16 else torch.int32)), nm
    none = idx.eq(-1).all(dim=2)
    assert bool((outs[0][0][none] == 0).all()) and bool(torch.isneginf(outs[0][1][none]).all()) and bool((outs[0][2][none] == 0).all())
