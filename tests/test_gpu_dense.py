"""The dense forward route: (query tile, KV block) pairs that at least half of a tile's tokens keep are computed by the
query-tile-outer kernel, everything else by the gather route.  Whatever the split, O and LSE match the oracle; the
split itself is found by counting (never assumed), so the cases here make the detection partial: ragged tiles, rows
that drop the sink, occupancy around the threshold, tiles at sequence starts, packed batches."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import nsa_sel_oracle as orc
from gpu_util import Case, TOL_GRAD, TOL_O, assert_close, assert_lse_close, to_f64

pytestmark = pytest.mark.gpu


def _check(w, window=0, expect_dense=None, bwd=False):
    Q, K, V, dO = (wl.bf16_bits_to_f64(x) for x in (w.q, w.k, w.v, w.do))
    rO, rL = orc.forward(Q, K, V, w.idx, w.cu_seqlens, causal=w.causal, block=w.block, window=window)
    frac = {}
    for dense in (True, False):
        c = Case(w, bwd=bwd, window=window, dense=dense)
        o, lse = c.forward()
        assert_close(f"O dense={dense}", to_f64(o), rO, TOL_O)
        assert_lse_close(to_f64(lse), rL)
        flags = c.attn.dense_entries()
        frac[dense] = float(flags.mean()) if flags.size else 0.0
        # the inversion result does not depend on the routing
        cnt, off, qlist, qslot, vmask, bcap = c.attn.index_arrays()
        rc, ro, rl, rs, rvm = orc.invert_index(w.idx, w.cu_seqlens, block=w.block, causal=w.causal, window=window)
        assert np.array_equal(cnt[:, :rc.shape[1]], rc) and np.array_equal(qlist, rl) and np.array_equal(qslot, rs)
        if bwd:
            dq, dk, dv = c.backward(o, lse)
            rq, rk, rv = orc.backward(Q, K, V, dO, w.idx, w.cu_seqlens, causal=w.causal, block=w.block, window=window)
            assert_close("dQ", to_f64(dq), rq, TOL_GRAD)
            assert_close("dK", to_f64(dk), rk, TOL_GRAD)
            assert_close("dV", to_f64(dv), rv, TOL_GRAD)
    assert frac[False] == 0.0
    print("  dense share of the pairs:", round(frac[True], 3), flush=True)
    if expect_dense is not None:
        lo, hi = expect_dense
        assert lo <= frac[True] <= hi, frac
    return frac[True]


@pytest.mark.parametrize("name", wl.SMALL_NAMES)
def test_both_routes_match_the_oracle(name):
    print("case dense/gather", name, flush=True)
    _check(wl.realise(wl.small(name)), bwd=name in ("g4", "g1_varlen", "b128_g4"))


@pytest.mark.parametrize("g,block,causal", [(1, 64, True), (3, 64, True), (5, 128, True), (8, 64, False), (2, 128, False)])
def test_tiles_of_one_piece_and_more(g, block, causal):
    """Every block kept by every token that sees it: causal, tiles of 1, 2, 3 .. pieces, the last one ragged; without the mask of an odd and
    of an even number."""
    print("case dense pieces", g, block, causal, flush=True)
    lengths = [block * 5 - 3] if causal else [block * 3 - 7, block, 4 * block - 1]
    w = wl.realise(wl.Workload("pieces", lengths, hq=2 * g, hkv=2, topk=8, causal=causal, block=block, sink=causal, seed=37))
    _check(w, expect_dense=(1.0, 1.0))


def test_sink_and_own_block_are_found_dense():
    """Sink + own block forced, 14 uniform picks: 2 of 16 slots of every late token, everything near the start."""
    print("case dense share", flush=True)
    w = wl.realise(wl.Workload("share", [4096], hq=8, hkv=2, topk=16, sink=True, seed=31))
    share = _check(w)
    assert 0.12 <= share <= 0.6


def test_rows_that_drop_the_sink_and_occupancy_around_the_threshold():
    print("case dense partial rows", flush=True)
    w = wl.realise(wl.Workload("partial", [1500, 700], hq=8, hkv=2, topk=8, sink=True, seed=32))
    rng = np.random.default_rng(5)
    T = w.total_tokens
    # every third token of the first KV head does not select the sink: the pair stays dense with a partial mask
    drop = (np.arange(T) % 3 == 0)
    w.idx[drop, 0, 0] = -1
    # tiles 8..15: block 2 kept by exactly 31, 32 or 33 of the 64 tokens (below, at and above one half)
    for n, tile in enumerate(range(8, 17)):
        keep = 31 + n % 3
        rows = np.arange(tile * 64, tile * 64 + 64)
        w.idx[rows, 1, 1] = np.where(np.arange(64) < keep, 2, w.idx[rows, 1, 1])
        clash = (w.idx[rows][:, 1, 2:] == 2).any(axis=1)            # keep rows duplicate-free for the recipe's sake
        w.idx[rows[clash], 1, 2:] = np.where(w.idx[rows[clash], 1, 2:] == 2, -1, w.idx[rows[clash], 1, 2:])
    # a tile whose first, middle and last tokens keep nothing at all
    w.idx[[1024, 1056, 1087], :, :] = -1
    _check(w, bwd=True)


def test_locality_picks_become_masked_dense_pairs():
    """Half of the free picks among the 8 most recent blocks (the g = 7 configuration's recipe): those pairs are kept
    by 7/8 of a tile's tokens and go dense with a row mask."""
    print("case dense locality", flush=True)
    w = wl.realise(wl.Workload("local", [3000], hq=7, hkv=1, topk=16, sink=True, local_picks=7, seed=33))
    share = _check(w, bwd=True)
    assert share >= 0.5


@pytest.mark.parametrize("seqlens,window,block", [([2000], 512, 64), ([700, 64, 1, 333, 1029], 100, 64),
                                                  ([900, 450], 300, 128), ([1500], 1, 64)])
def test_window_branch_is_all_dense(seqlens, window, block):
    print("case dense window", seqlens, window, block, flush=True)
    w = wl.realise(wl.Workload("win", seqlens, hq=4, hkv=2, topk=1, block=block, seed=34))
    w.idx = wl.window_block_indices(seqlens, 2, window, block)
    w.topk = w.idx.shape[2]
    _check(w, window=window, expect_dense=(0.9, 1.0), bwd=True)


def test_adversarial_selections_and_empty_rows():
    print("case dense adversarial", flush=True)
    w = wl.realise(wl.Workload("adv", [900, 300, 0, 65], hq=6, hkv=2, topk=10, seed=23))
    w.idx = wl.draw_adversarial_indices(np.random.default_rng(4), w.seqlens, w.hkv, w.topk)
    w.idx[100:140] = -1
    _check(w, bwd=True)
    w2 = wl.realise(wl.Workload("nc", [700, 300], hq=4, hkv=2, topk=12, causal=False, seed=35))
    w2.idx[:, :, 0] = 1                                            # every token of both sequences selects block 1
    _check(w2)


def test_dense_route_with_capped_workspace_is_bit_identical():
    print("case dense capped ws", flush=True)
    import paper_2508_18224_amd as nsa
    w = wl.realise(wl.small("g2_hkv5"))
    c = Case(w, bwd=False)
    o, lse = c.forward()
    c.attn = nsa.SelAttention(w.total_tokens, w.hq, w.hkv, w.topk, nseq=len(w.seqlens), causal=w.causal,
                              block=w.block, ws_cap_bytes=1, bwd=False, dense=True)
    o2, lse2 = c.forward()
    assert c.attn.dense_entries().any()
    assert torch.equal(o, o2) and torch.equal(lse, lse2)


def test_default_routing_policy():
    """shape.dense = 0: the dense route where it pays (g >= 2, or a window), the gather route at g = 1."""
    print("case dense policy", flush=True)
    import paper_2508_18224_amd as nsa
    big = wl.Workload("policy_g2", [9000], hq=4, hkv=2, topk=16, sink=True, seed=41)      # 288K triples
    big1 = wl.Workload("policy_g1", [9000, 300], hq=2, hkv=2, topk=16, seed=42)
    for name, window, expect in ((big, 0, True), (big1, 0, False), (big1, 100, True), ("g4", 0, False)):
        w = wl.realise(wl.small(name) if isinstance(name, str) else name)
        c = Case(w, bwd=False, window=window)
        c.attn = nsa.SelAttention(w.total_tokens, w.hq, w.hkv, w.topk, nseq=len(w.seqlens), causal=w.causal,
                                  block=w.block, window=window, bwd=False)        # dense=None: the library picks
        c.forward()
        assert bool(c.attn.dense_entries().any()) == expect, (name, window)


@pytest.mark.parametrize("step", [0.5, 6.0, 10.0])
def test_climbing_maxima_and_independence_of_the_other_rows(step):
    """The running maximum of every second token climbs by `step` (log2 domain) from piece to piece, that of its neighbours
    stays flat: the result matches the oracle, and a row's bits do not depend on the rows it shares a wavefront with."""
    print("case dense climbing maxima", step, flush=True)
    T, window = 1024, 512
    w = wl.realise(wl.Workload("climb", [T], hq=2, hkv=1, topk=1, seed=36))
    w.idx = wl.window_block_indices([T], 1, window)                # the most recent block first: pieces go back in time
    w.topk = w.idx.shape[2]
    q, k = wl.bf16_bits_to_f32(w.q).copy(), wl.bf16_bits_to_f32(w.k).copy()
    # channel 0 carries the climb: older blocks score higher by `step` / (scale log2 e) for a query of 1 there
    level = step / (1.4426950408889634 * 128 ** -0.5)
    k[:, :, 0] = level / 16 * (T // 64 - np.arange(T) // 64)[:, None]
    q *= 0.25
    q[0::2, :, 0], q[1::2, :, 0] = 16.0, 0.0
    w.q, w.k = wl.f32_to_bf16_bits(q), wl.f32_to_bf16_bits(k)
    _check(w, window=window, expect_dense=(0.9, 1.0))
    o, lse = Case(w, bwd=False, window=window).forward()
    q[1::2, :, 0] = 48.0                                           # now the neighbours climb three times as fast
    w.q = wl.f32_to_bf16_bits(q)
    _check(w, window=window)
    o2, lse2 = Case(w, bwd=False, window=window).forward()
    assert torch.equal(o[0::2], o2[0::2]) and torch.equal(lse[0::2], lse2[0::2])
    assert not torch.equal(o[1::2], o2[1::2])


@pytest.mark.parametrize("block,dense", [(64, True), (128, True), (64, False), (128, False)])
def test_rows_past_a_ragged_block_are_never_used(block, dense):
    """Short ragged blocks of packed sequences with several KV heads: NaN in the K and V of every second sequence and behind
    the last token leaves the results of the other sequences as they are, bit for bit - a masked key still meets its V row
    as 0 * V, so one foreign row would show."""
    print("case dense ragged guard", block, dense, flush=True)
    seqlens = [65, 70, 1, 85, 17, 112, 130, 33, 81]
    w = wl.realise(wl.Workload("guard", seqlens, hq=4, hkv=2, topk=4, block=block, sink=True, seed=37))
    T = w.total_tokens
    seq = torch.from_numpy(np.repeat(np.arange(len(seqlens)), seqlens)).cuda()
    c = Case(w, dense=dense)
    rO, rL = orc.forward(*c.host_f64()[:3], w.idx, w.cu_seqlens, block=block)
    o0, lse0 = c.forward()
    g0 = c.backward(o0, lse0)
    assert_close("O", to_f64(o0), rO, TOL_O)
    if dense:
        assert c.attn.dense_entries().any()
    clean = (c.k, c.v)
    for bad in (0, 1):
        padded = []
        for x in clean:
            p = torch.full((T + 128, 2, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
            p[:T] = x
            p[:T][seq % 2 == bad] = float("nan")
            padded.append(p)
        c.k, c.v = padded[0][:T], padded[1][:T]
        o, lse = c.forward()
        grads = c.backward(o, lse)
        good = seq % 2 != bad
        assert torch.equal(o[good], o0[good]) and torch.equal(lse[good], lse0[good]) and bool(torch.isfinite(o[good]).all())
        for a, b in zip(grads, g0):
            assert torch.equal(a[good], b[good])


@pytest.mark.parametrize("topk,sink", [(2, False), (6, True), (9, True), (10, True), (10, False), (17, False), (19, True), (26, True),
                                       (27, False), (32, False)])
def test_rounds_of_gathered_columns(topk, sink):
    """The columns that are not dense (all but the own block and, with a sink, block 0) are gathered in rounds of like size, four to
    eight columns each: one round (four of them in part empty), a full one, two, three and four."""
    print("case rounds", topk, sink, flush=True)
    _check(wl.realise(wl.Workload("rounds", [2560, 61], hq=2, hkv=1, topk=topk, sink=sink, seed=59)))


def test_a_row_does_not_depend_on_its_neighbours():
    """Odd tokens keep the same blocks in both selections, even ones up to twenty more in the second, none of them dense: the partial
    rows of a wavefront are gathered in rounds that differ in length, and the odd tokens' bits are the same."""
    print("case neighbours", flush=True)
    tokens, hkv, topk = 8192, 2, 32
    w = wl.realise(wl.Workload("neighbours", [tokens], hq=4, hkv=hkv, topk=topk, sink=True, seed=61))
    c = Case(w, bwd=False, dense=True)
    keep = np.random.default_rng(2).integers(5, 18, size=(tokens, hkv))
    column = np.arange(topk)[None, None, :]
    outs = []
    for more in (0, 1):
        idx = w.idx.copy()
        kept = np.where((np.arange(tokens) % 2 == 0)[:, None], keep + more * np.random.default_rng(3).integers(0, 21, size=keep.shape), keep)
        idx[column >= kept[..., None]] = -1
        c.idx = torch.from_numpy(idx).cuda()
        o, lse = c.forward()
        assert c.attn.dense_entries().any()
        outs.append((o[6145::2].clone(), lse[6145::2].clone()))    # (earlier tiles have few blocks: what is dense there differs)
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])


@pytest.mark.parametrize("dense", [True, None])
def test_the_largest_probability_is_exact(dense):
    """Wide scores, whose rows are carried by few keys: against the running maximum the largest probability is 1, which bf16 holds, and what
    is left of O's error is little more than its own rounding to bf16 (1.04 and 1.03 times that; 1.26 and 1.22 against a maximum that was
    let lag behind).  With every probability rounded, two independent errors of a size, it would be 1.4 times."""
    print("case largest probability", dense, flush=True)
    w = wl.realise(wl.Workload("wide", [1500], hq=8, hkv=2, topk=1, seed=39), tensors=True)
    w.idx = wl.window_block_indices(w.seqlens, w.hkv, 512, 64)
    w.topk = w.idx.shape[2]
    c = Case(w, bwd=False, window=512, dense=dense)
    c.q *= 4
    o, lse = c.forward()
    rO, rL = orc.forward(to_f64(c.q), to_f64(c.k), to_f64(c.v), w.idx, w.cu_seqlens, window=512)
    rounding = np.linalg.norm(to_f64(torch.from_numpy(rO).bfloat16()) - rO)
    ratio = np.linalg.norm(to_f64(o) - rO) / rounding
    print("  error over that of rounding O", round(ratio, 3), flush=True)
    assert ratio < 1.1
    assert np.abs(to_f64(lse) - rL).max() < 2e-5  # 32-bit sums and a maximum of some tens
