"""The forward of short inputs (k_fwd_short), which the library picks by itself (shape.dense = 0), against the oracle and against the
gather route (shape.dense = -1): every form of input it takes over, at the edges of its row groups, pieces and splits."""
import numpy as np
import pytest
import torch

import paper_2508_18224_amd as nsa
import workloads as wl
from oracle import nsa_sel_oracle as orc
from gpu_util import Case, TOL_O, assert_close, assert_lse_close, to_f64

pytestmark = pytest.mark.gpu


def _attn(w, window=0, dense=None, cap=None):
    return nsa.SelAttention(w.total_tokens, w.hq, w.hkv, w.topk, nseq=len(w.seqlens), causal=w.causal, block=w.block, window=window,
                            ws_cap_bytes=cap, dense=dense)


def _kinds(call):
    nsa.binding.profile_enable(64)
    try:
        out = call()
        torch.cuda.synchronize()
        return out, {k for k, (_, n) in nsa.binding.profile_collect().items() if n}
    finally:
        nsa.binding.profile_enable(0)


def _check(w, window=0, backward=True):
    c = Case(w, window=window)
    short, gather = _attn(w, window), _attn(w, window, dense=False)
    short.index_ws.fill_(0x5A)
    (o, lse), kinds = _kinds(lambda: short.forward(c.q, c.k, c.v, c.idx, c.cu))
    assert "fwd_short" in kinds and not kinds & {"fwd_main", "fwd_merge", "fwd_dense"}, kinds
    Q, K, V, _ = c.host_f64()
    rO, rL = orc.forward(Q, K, V, w.idx, w.cu_seqlens, causal=w.causal, block=w.block, window=window)
    assert_close("O", to_f64(o), rO, TOL_O)
    assert_lse_close(to_f64(lse), rL)
    # the error is no larger than the gather route's, whose partial rows are rounded to bf16
    o_g, lse_g = gather.forward(c.q, c.k, c.v, c.idx, c.cu)
    assert np.linalg.norm(to_f64(o) - rO) <= 1.02 * np.linalg.norm(to_f64(o_g) - rO) + 1e-9
    # the index it leaves is the inversion's, bit for bit, and so are the gradients from it
    for a, b in zip(short.index_arrays()[:5], gather.index_arrays()[:5]):
        assert np.array_equal(a, b)
    if backward:
        for a, b in zip(short.backward(c.q, c.k, c.v, o_g, lse_g, c.do, c.cu), gather.backward(c.q, c.k, c.v, o_g, lse_g, c.do, c.cu)):
            assert torch.equal(a, b)
    # from the index alone, with a capped workspace, and twice: the same bits
    again = [short.forward(c.q, c.k, c.v, None, c.cu, rebuild_index=False), short.forward(c.q, c.k, c.v, c.idx, c.cu),
             _attn(w, window, cap=1).forward(c.q, c.k, c.v, c.idx, c.cu)]
    for o2, lse2 in again:
        assert torch.equal(o, o2) and torch.equal(lse, lse2)
    return c, o, lse


@pytest.mark.parametrize("seqlens,g,hkv,topk,block", [
    ([1], 1, 1, 1, 64), ([63], 8, 1, 1, 64), ([64, 65], 2, 2, 2, 64), ([129, 1, 0, 127, 128], 1, 3, 4, 64), ([1000], 4, 1, 8, 64),
    ([900, 300], 7, 2, 7, 64), ([2000], 4, 8, 16, 64), ([700, 64, 1, 333, 0], 3, 2, 10, 64), ([1500, 37], 5, 1, 32, 64),
    ([1100], 8, 2, 32, 128), ([257, 128, 1, 515], 2, 2, 9, 128), ([2500], 1, 2, 16, 64),
    ([4096], 1, 32, 16, 64)])  # the last: more counters than the scatter folds in, their prefix is a launch of its own
def test_short_forward_matches_oracle(seqlens, g, hkv, topk, block):
    print("case short", seqlens, g, hkv, topk, block, flush=True)
    w = wl.realise(wl.Workload("short", seqlens, hq=g * hkv, hkv=hkv, topk=topk, block=block, sink=topk > 2, seed=81))
    _check(w)


@pytest.mark.parametrize("seed", range(4))
def test_short_forward_adversarial_and_bidirectional_rows(seed):
    """Future, foreign, repeated and padded ids, and rows with nothing visible, in both directions."""
    rng = np.random.default_rng(90 + seed)
    seqlens = [int(x) for x in rng.integers(1, 170, size=int(rng.integers(1, 4)))]
    block, hkv, g, topk = int(rng.choice([64, 128])), int(rng.integers(1, 4)), int(rng.integers(1, 9)), int(rng.choice([8, 11, 32]))
    print("case short adversarial", seed, seqlens, block, hkv, g, topk, flush=True)
    w = wl.realise(wl.Workload("adv", seqlens, hq=g * hkv, hkv=hkv, topk=topk, causal=bool(seed % 2), block=block, seed=seed))
    w.idx = wl.draw_adversarial_indices(rng, seqlens, hkv, topk, block=block)
    w.idx[:: 7] = -1
    _check(w)


@pytest.mark.parametrize("window,block,tokens", [(1, 64, 200), (100, 64, 1000), (129, 128, 700), (512, 64, 3000), (1000, 64, 2500)])
def test_short_forward_windows(window, block, tokens):
    print("case short window", window, block, tokens, flush=True)
    w = wl.realise(wl.Workload("win", [tokens, 90], hq=4, hkv=2, topk=1, block=block, seed=83), tensors=True)
    w.idx = wl.window_block_indices(w.seqlens, w.hkv, window, block)
    w.topk = w.idx.shape[2]
    _check(w, window=window)


def test_longest_input_and_where_the_choice_ends():
    """8192 tokens (128 pieces a sequence) go this way where top-k is large, 8193 tokens and small top-k do not."""
    print("case short limits", flush=True)
    for tokens, topk, hq, expect in ((8192, 32, 8, True), (8193, 32, 8, False), (8192, 16, 8, False), (3000, 16, 8, True), (4096, 16, 8, False)):
        w = wl.realise(wl.Workload("limit", [tokens], hq=hq, hkv=1, topk=topk, sink=True, seed=84))
        c = Case(w, bwd=False)
        (o, lse), kinds = _kinds(lambda: _attn(w).forward(c.q, c.k, c.v, c.idx, c.cu))
        assert ("fwd_short" in kinds) == expect, (tokens, topk, kinds)
        o_g, lse_g = _attn(w, dense=False).forward(c.q, c.k, c.v, c.idx, c.cu)
        assert float((o.float() - o_g.float()).norm() / o_g.float().norm()) < 6e-3  # bf16 probabilities and partial rows
        assert float((lse - lse_g).abs().max()) < 1e-4


@pytest.mark.parametrize("tokens,hq,hkv", [(600, 4, 2), (2000, 32, 8)])
def test_foreign_infinities_and_neighbours_do_not_show(tokens, hq, hkv):
    """NaN and infinities in the K and V of two blocks: rows that keep neither have the bits they have without them, rows that do are
    not finite.  And a row's bits do not depend on what the other tokens of its group keep."""
    print("case short isolation", tokens, hq, hkv, flush=True)
    w = wl.realise(wl.Workload("iso", [tokens], hq=hq, hkv=hkv, topk=10, sink=False, seed=85))
    c, attn = Case(w, bwd=False), _attn(w)
    o, lse = attn.forward(c.q, c.k, c.v, c.idx, c.cu)
    k, v = c.k.clone(), c.v.clone()
    k[64:128], v[64:128], v[256:320] = float("nan"), float("inf"), float("-inf")
    o_bad, lse_bad = attn.forward(c.q, k, v, c.idx, c.cu)
    kept = torch.from_numpy(((w.idx == 1) | (w.idx == 4)).any(axis=2)).cuda().repeat_interleave(hq // hkv, dim=1)
    assert bool(kept.any()) and not bool(kept.all())
    assert torch.equal(o_bad[~kept], o[~kept]) and torch.equal(lse_bad[~kept], lse[~kept])
    assert not bool(torch.isfinite(o_bad.float())[kept].all(dim=-1).any())
    idx = c.idx.clone()
    idx[1::2, :, 3:] = -1                              # every other token keeps less
    o_less, lse_less = attn.forward(c.q, c.k, c.v, idx, c.cu)
    assert torch.equal(o_less[0::2], o[0::2]) and torch.equal(lse_less[0::2], lse[0::2])


@pytest.mark.parametrize("tokens,hq,hkv,window,block", [(600, 4, 2, 0, 64), (2000, 32, 8, 0, 64), (1100, 8, 4, 300, 64), (700, 8, 2, 0, 128)])
def test_scores_of_minus_infinity(tokens, hq, hkv, window, block):
    """Keys masked with -inf in K: rows whose first pieces score -inf throughout, rows that meet such a piece behind a finite one, and
    rows that see nothing else, whose LSE is -inf and whose O is not a number, as by every other route."""
    print("case short -inf scores", tokens, hq, hkv, window, block, flush=True)
    if window:
        w = wl.realise(wl.Workload("masked", [tokens], hq=hq, hkv=hkv, topk=1, block=block, seed=91), tensors=True)
        w.idx = wl.window_block_indices(w.seqlens, w.hkv, window, block)
        w.topk = w.idx.shape[2]
    else:
        w = wl.realise(wl.Workload("masked", [tokens], hq=hq, hkv=hkv, topk=8, block=block, sink=True, seed=91))
    c = Case(w, window=window)
    c.q[..., 0] = c.q[..., 0].abs() + 0.125
    c.k[:128, :, 0] = float("-inf")          # the first pieces of the sequence, and one within it
    c.k[384:448, :, 0] = float("-inf")
    gate = torch.from_numpy(wl.draw_gates(w.seed, w.total_tokens, w.hq)).cuda()
    attn = _attn(w, window)
    (out, o, lse), kinds = _kinds(lambda: attn.forward_gated(c.q, c.k, c.v, c.idx, gate, c.do, c.cu))
    assert "fwd_short" in kinds
    with np.errstate(invalid="ignore", divide="ignore"):
        rO, rL = orc.forward(to_f64(c.q), to_f64(c.k), to_f64(c.v), w.idx, w.cu_seqlens, block=block, window=window)
    lost = ~np.isfinite(rL)                  # everything such a row sees is masked
    assert lost.any() and not lost.all() and np.isnan(rO[lost]).all()
    assert_close("O", to_f64(o)[~lost], rO[~lost], TOL_O)
    assert np.abs(to_f64(lse) - rL)[~lost].max() <= 1e-3
    assert np.isneginf(to_f64(lse)[lost]).all() and np.isnan(to_f64(o)[lost]).all() and np.isnan(to_f64(out)[lost]).all()
    assert np.isfinite(to_f64(out)[~lost]).all()
    # the dense route says the same (the partial rows of the gather route, of which a window leaves none, are not numbers there)
    o_d, lse_d = _attn(w, window, dense=True).forward(c.q, c.k, c.v, c.idx, c.cu)
    assert torch.equal(torch.isneginf(lse_d), torch.isneginf(lse)) and bool(torch.isfinite(lse_d)[torch.isfinite(lse)].all())
    if window:
        assert torch.equal(torch.isnan(o_d), torch.isnan(o))


@pytest.mark.parametrize("dense", [None, True])
def test_scale_next_to_nothing(dense):
    """A scale whose reciprocal times eight is infinite in fp32: every visible key counts the same."""
    print("case short scale", dense, flush=True)
    w = wl.realise(wl.Workload("flat", [500, 90], hq=4, hkv=2, topk=6, sink=True, seed=92))
    c = Case(w, bwd=False, scale=1e-38, dense=dense)
    o, lse = c.forward()
    Q, K, V, _ = c.host_f64()
    rO, rL = orc.forward(Q, K, V, w.idx, w.cu_seqlens, scale=1e-38)
    assert_close("O", to_f64(o), rO, TOL_O)
    assert_lse_close(to_f64(lse), rL)


def test_short_gated_forward():
    print("case short gated", flush=True)
    w = wl.realise(wl.Workload("gated", [800, 130], hq=6, hkv=2, topk=8, sink=True, seed=86))
    c = Case(w)
    gate = torch.from_numpy(wl.draw_gates(w.seed, w.total_tokens, w.hq)).cuda()
    acc = torch.randn_like(c.q.float()).bfloat16()
    attn = _attn(w)
    o, lse = attn.forward(c.q, c.k, c.v, c.idx, c.cu)
    (out, o2, lse2), kinds = _kinds(lambda: attn.forward_gated(c.q, c.k, c.v, c.idx, gate, acc, c.cu))
    assert "fwd_short" in kinds and torch.equal(o, o2) and torch.equal(lse, lse2)
    want = acc.double() + gate.double()[..., None] * o.double()
    assert_close("O_out", to_f64(out), to_f64(want), TOL_O)
    buf = acc.clone()
    in_place, _, _ = attn.forward_gated(c.q, c.k, c.v, c.idx, gate, buf, c.cu, out=buf)
    assert torch.equal(in_place, out)


def test_short_step_replays_from_a_hip_graph():
    print("case short graph", flush=True)
    ws = [wl.realise(wl.Workload("graph", [900, 77], hq=4, hkv=2, topk=8, sink=True, seed=s)) for s in (87, 88)]
    refs = []
    for w in ws:
        c = Case(w)
        refs.append(_attn(w).forward(c.q, c.k, c.v, c.idx, c.cu))
    c, attn = Case(ws[0]), _attn(ws[0])
    o, lse = (torch.empty_like(x) for x in refs[0])
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        attn.forward(c.q, c.k, c.v, c.idx, c.cu, out=o, lse=lse)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        attn.forward(c.q, c.k, c.v, c.idx, c.cu, out=o, lse=lse)
    for rep in (1, 0, 1):
        d = Case(ws[rep])
        for dst, src in ((c.q, d.q), (c.k, d.k), (c.v, d.v), (c.idx, d.idx)):
            dst.copy_(src)
        attn.index_ws.fill_(0x5A)
        o.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(o, refs[rep][0]) and torch.equal(lse, refs[rep][1])
