"""Capped workspaces (buffer reuse over head subsets, paper App. E): with a workspace that holds only some
of the KV heads the library works through the heads in several passes; the results must be bit-identical to
the single-pass ones (same arithmetic, same order) and the forward must still match the oracle."""
import numpy as np
import pytest
import torch

import paper_2508_18224_amd as nsa
import workloads as wl
from gpu_util import Case, TOL_O, assert_close, assert_lse_close, to_f64
from oracle import nsa_sel_oracle as oracle

pytestmark = pytest.mark.gpu


def _run(case):
    o, lse = case.forward()
    dq, dk, dv = case.backward(o, lse)
    return [x.clone() for x in (o, lse, dq, dk, dv)]


def _same_bits(a, b):
    if a.dtype == torch.bfloat16:
        return torch.equal(a.view(torch.int16), b.view(torch.int16))
    return torch.equal(a.view(torch.int32), b.view(torch.int32))


@pytest.mark.parametrize("name,heads", [("g2_hkv5", 1), ("g2_hkv5", 2), ("g1_varlen", 1), ("b128_g4", 1)])
def test_capped_workspace_matches_single_pass(name, heads):
    w = wl.realise(wl.small(name))
    full = Case(w)
    ref = _run(full)
    fmin, bmin = nsa.workspace_bytes_min(full.attn.shape)
    ffull, bfull, _ = nsa.workspace_bytes(full.attn.shape)
    assert fmin < ffull and bmin < bfull
    capped = Case(w)
    capped.attn = nsa.SelAttention(w.total_tokens, w.hq, w.hkv, w.topk, nseq=len(w.seqlens), causal=w.causal,
                                   block=w.block, ws_cap_bytes=heads * max(fmin, bmin), dense=True)
    assert capped.attn.fwd_ws.numel() < ffull and capped.attn.bwd_ws.numel() < bfull
    # poison the reused buffers so that a stale read from an earlier pass cannot go unnoticed
    capped.attn.fwd_ws.fill_(0x7F)
    capped.attn.bwd_ws.fill_(0x7F)
    got = _run(capped)
    for nm, a, b in zip(("O", "LSE", "dQ", "dK", "dV"), got, ref):
        assert _same_bits(a, b), f"{nm} differs between the capped and the full workspace"
    q, k, v, _ = full.host_f64()
    o_ref, lse_ref = oracle.forward(q, k, v, w.idx, w.cu_seqlens, block=w.block, causal=w.causal)
    assert_close("O", to_f64(got[0]), o_ref, TOL_O)
    assert_lse_close(to_f64(got[1]), lse_ref)


def test_workspace_below_minimum_is_rejected():
    w = wl.realise(wl.small("g2_hkv5"))
    case = Case(w)
    fmin, bmin = nsa.workspace_bytes_min(case.attn.shape)
    case.attn.fwd_ws = torch.empty(fmin - 256, dtype=torch.uint8, device="cuda")
    with pytest.raises(nsa.NsaSelError):
        case.forward()


@pytest.mark.parametrize("seqlens,hq,hkv,topk", [([1024], 4, 1, 8), ([2000], 8, 2, 16), ([700, 1, 333], 16, 2, 4),
                                                 ([1200], 8, 1, 3), ([2000], 2, 1, 16)])
def test_capped_workspace_of_tiny_inputs_matches_single_pass(seqlens, hq, hkv, topk):
    """The smaller work units of tiny inputs have more dK/dV sums than the smallest backward workspace holds: the KV blocks
    of a head are gone through in ranges, with the same units and so the same bits."""
    print("case capped tiny", seqlens, hq, hkv, topk, flush=True)
    w = wl.realise(wl.Workload("tiny_cap", seqlens, hq=hq, hkv=hkv, topk=topk, sink=True, seed=93))
    full = Case(w)
    ref = _run(full)
    _, bmin = nsa.workspace_bytes_min(full.attn.shape)
    one_head = nsa.Shape.from_buffer_copy(full.attn.shape)
    one_head.unit = 256
    assert bmin <= nsa.workspace_bytes_min(one_head)[1]
    for cap in (bmin, bmin + 5 * 65536):
        capped = Case(w)
        capped.attn = nsa.SelAttention(w.total_tokens, w.hq, w.hkv, w.topk, nseq=len(w.seqlens), ws_cap_bytes=cap, dense=True)
        assert capped.attn.shape.unit == 0 and capped.attn.bwd_ws.numel() == cap < full.attn.bwd_ws.numel()
        capped.attn.bwd_ws.fill_(0x7F)
        for nm, a, b in zip(("O", "LSE", "dQ", "dK", "dV"), _run(capped), ref):
            assert _same_bits(a, b), f"{nm} differs between the capped and the full workspace"


@pytest.mark.parametrize("tokens,block", [(9900, 64), (9990, 128)])
def test_reduction_by_ranges_of_lists_matches_one_list_each(tokens, block):
    """The dK/dV reduction gives a workgroup lists x block / 4 / 4096 lists: three of 775 (of 395 blocks of 128 tokens)
    with all KV heads in one pass, the last range short, and one of 155 (79) with a KV head per pass.  Same bits."""
    print("case list ranges", tokens, block, flush=True)
    w = wl.realise(wl.Workload("ranges", [tokens], hq=5, hkv=5, topk=4, block=block, sink=True, seed=95))
    lists = 5 * (tokens // block + 1)
    per = lists * (block // 4) // 4096
    assert per == 3 and lists % per and lists // 5 * (block // 4) < 2 * 4096
    full = Case(w)
    ref = _run(full)
    capped = Case(w)
    capped.attn = nsa.SelAttention(tokens, 5, 5, 4, block=block, ws_cap_bytes=1, dense=True)
    capped.attn.bwd_ws.fill_(0x7F)
    for nm, a, b in zip(("O", "LSE", "dQ", "dK", "dV"), _run(capped), ref):
        assert _same_bits(a, b), nm


@pytest.mark.parametrize("seqlens,hq,hkv,topk,block,dense", [([8201], 32, 32, 5, 64, False), ([3000, 1, 5200], 33, 11, 17, 64, False),
                                                             ([9001], 30, 6, 32, 128, False), ([9001], 30, 6, 3, 64, True)])
def test_reduction_in_bursts_matches_row_by_row(seqlens, hq, hkv, topk, block, dense):
    """From 2^17 rows a pass and eight columns on the dQ reduction writes a workgroup's rows at once, else as they are done: one pass takes
    the former with 17 and 32 columns (the last workgroup of it part empty), a KV head per pass and fewer columns the latter.  Same sums
    in the same order, same bits; gated and plain, more and fewer columns than a batch.  (The merge in bursts: test_gpu_reductions.py.)"""
    print("case bursts", seqlens, hq, hkv, topk, block, dense, flush=True)
    w = wl.realise(wl.Workload("bursts", seqlens, hq=hq, hkv=hkv, topk=topk, block=block, sink=True, seed=96))
    rows = w.total_tokens * hq
    assert rows >= 1 << 18 and rows % 512 and rows // hkv < 1 << 18
    gen = torch.Generator(device="cuda").manual_seed(7)
    gate = torch.rand(w.total_tokens, hq, generator=gen, device="cuda")
    gate[::7] = 0
    acc = torch.randn(w.total_tokens, hq, 128, generator=gen, device="cuda").to(torch.bfloat16)
    outs = []
    for cap in (None, 1):
        case = Case(w)
        case.attn = nsa.SelAttention(w.total_tokens, hq, hkv, topk, nseq=len(seqlens), block=block, ws_cap_bytes=cap, dense=dense)
        for ws in (case.attn.fwd_ws, case.attn.bwd_ws):
            ws.fill_(0x7F)
        got = _run(case)
        case.attn.fwd_ws.fill_(0x7F)
        got += [x.clone() for x in case.attn.forward_gated(case.q, case.k, case.v, case.idx, gate, acc, case.cu)]
        outs.append(got)
    for nm, a, b in zip(("O", "LSE", "dQ", "dK", "dV", "gated O_out", "gated O", "gated LSE"), *outs):
        assert _same_bits(a, b), nm
    assert _same_bits(outs[0][0], outs[0][6]) and _same_bits(outs[0][1], outs[0][7])
    plain = acc.float() + gate[..., None] * outs[0][0].float()
    # two bf16 roundings apart: the library adds the sum before it is rounded
    assert ((outs[0][5].float() - plain).abs() <= 2.0 ** -7 * (plain.abs() + outs[0][0].float().abs())).all()
