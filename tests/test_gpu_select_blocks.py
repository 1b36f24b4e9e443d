"""Block selection on the GPU (scores -> selection tensor) must equal the oracle's bit for bit: the decision is
taken on the fp32 scores as given on both sides, and the tie rule makes every row unique."""
import ctypes as C

import numpy as np
import pytest
import torch

import paper_2508_18224_amd as nsa
import workloads as wl
from oracle import nsa_sel_oracle as orc
from oracle import topk_select_oracle as tko

pytestmark = pytest.mark.gpu


def _cu(seqlens):
    return np.concatenate([[0], np.cumsum(seqlens)]).astype(np.int32)


def _gpu_select(x, cu, topk, **kw):
    out = nsa.select_blocks(torch.from_numpy(x).cuda(), None if cu is None else torch.from_numpy(cu).cuda(), topk, **kw)
    torch.cuda.synchronize()
    return out.cpu().numpy()


@pytest.mark.parametrize("seqlens,hkv,topk,block,causal,n_sink,n_local,kind,stride", [
    ([2000], 2, 16, 64, True, 1, 2, "heavy", None),            # rows of 1 .. 32 blocks, 16-byte loads
    ([2000], 2, 16, 64, True, 1, 2, "ties", 33),               # odd stride: 4-byte loads
    ([700, 64, 1, 333, 1029], 3, 16, 64, True, 1, 2, "wild", None),
    ([900, 450], 2, 8, 64, False, 1, 1, "wild", 16),
    ([2100], 2, 8, 128, True, 1, 2, "ties", None),
    ([700, 129, 128, 1, 515], 2, 4, 128, True, 0, 1, "heavy", None),
    ([1500], 1, 32, 64, True, 2, 3, "ties", 24),
    ([777], 1, 1, 64, True, 0, 1, "heavy", None),
    ([777], 1, 1, 64, True, 0, 0, "heavy", None),
    ([1300], 2, 3, 64, True, 3, 3, "ties", None),              # more forced blocks than columns
    ([1300], 2, 12, 64, False, 0, 0, "wild", 21),              # plain top-k
])
def test_selection_bit_exact(seqlens, hkv, topk, block, causal, n_sink, n_local, kind, stride):
    print("case", seqlens, hkv, topk, block, causal, n_sink, n_local, kind, stride, flush=True)
    cu = _cu(seqlens)
    x = wl.draw_block_scores(31, seqlens, hkv, block, kind=kind, stride=stride, trap_future=causal)
    ref = tko.select_blocks(x, cu, topk, block=block, causal=causal, n_sink=n_sink, n_local=n_local)
    got = _gpu_select(x, cu, topk, block=block, causal=causal, n_sink=n_sink, n_local=n_local)
    assert np.array_equal(got, ref)


def test_single_sequence_without_cu():
    print("case no cu", flush=True)
    x = wl.draw_block_scores(32, [1000], 2, kind="heavy")
    ref = tko.select_blocks(x, _cu([1000]), 8)
    assert np.array_equal(_gpu_select(x, None, 8), ref)


@pytest.mark.parametrize("n_tokens,causal,kind,stride", [(70000, True, "ties", None), (140000, False, "heavy", 2190),
                                                         (140000, True, "ties", 2189)])
def test_rows_longer_than_one_chunk(n_tokens, causal, kind, stride):
    """More than 1024 visible blocks: the picks of several chunks are merged.  Oracle on sampled rows."""
    print("case multi-chunk", n_tokens, causal, kind, stride, flush=True)
    seqlens = [n_tokens]
    cu = _cu(seqlens)
    x = wl.draw_block_scores(33, seqlens, 1, kind=kind, stride=stride, trap_future=causal)
    rng = np.random.default_rng(5)
    tokens = np.unique(np.concatenate([rng.integers(0, n_tokens, 150), [0, 63, 64, 65535, 65536, 65599, 65600,
                                                                        n_tokens - 1]]))
    ref = tko.select_blocks(x, cu, 16, causal=causal, tokens=tokens)
    got = _gpu_select(x, cu, 16, causal=causal)
    assert np.array_equal(got[tokens], ref[tokens])


@pytest.mark.parametrize("n_tokens,causal,fill", [(70000, False, 0.25), (140000, True, -np.inf), (3000, True, np.nan)])
def test_all_scores_equal(n_tokens, causal, fill):
    """Every score the same: the bound the fast method derives keeps every block, so the row is handed to the general
    method (in rows of more than 128 blocks); the picks are then the smallest selectable block ids."""
    print("case all equal", n_tokens, causal, fill, flush=True)
    seqlens = [n_tokens]
    cu = _cu(seqlens)
    nb = -(-n_tokens // 64)
    x = np.full((n_tokens, 1, nb), fill, dtype=np.float32)
    rng = np.random.default_rng(7)
    tokens = np.unique(np.concatenate([rng.integers(0, n_tokens, 120), [0, 64, 2047, 2048, n_tokens - 1]]))
    ref = tko.select_blocks(x, cu, 16, causal=causal, tokens=tokens)
    got = _gpu_select(x, cu, 16, causal=causal)
    assert np.array_equal(got[tokens], ref[tokens])
    last = ref[n_tokens - 1, 0].tolist()
    assert last[:3] == ([0, (n_tokens - 1) // 64, (n_tokens - 1) // 64 - 1]) and last[3:] == list(range(1, 14))


def test_many_ties_at_the_bound():
    """A few distinct large scores over a sea of equal ones: more picks than distinct values, so the last picks are
    decided by block id among hundreds of equal scores."""
    print("case ties at the bound", flush=True)
    n_tokens, hkv = 100000, 2
    seqlens = [60000, 40000]
    cu = _cu(seqlens)
    rng = np.random.default_rng(8)
    x = np.ones((n_tokens, hkv, 938), dtype=np.float32)
    hot = rng.integers(0, 938, size=(n_tokens, hkv, 6))
    np.put_along_axis(x, hot, rng.random((n_tokens, hkv, 6)).astype(np.float32) + 2, axis=2)
    tokens = np.unique(np.concatenate([rng.integers(0, n_tokens, 150), [59999, 60000, n_tokens - 1]]))
    for causal in (True, False):
        ref = tko.select_blocks(x, cu, 16, causal=causal, tokens=tokens)
        got = _gpu_select(x, cu, 16, causal=causal)
        assert np.array_equal(got[tokens], ref[tokens])


def test_headline_shape_sampled_rows_and_properties():
    """N = 64K, 8 KV heads, 1024 blocks per row, top-16 with the sink and two local blocks forced: sampled rows
    against the oracle, and on every row the properties that hold at any size."""
    print("case headline selection", flush=True)
    T, hkv, topk = 65536, 8, 16
    seqlens = [T]
    cu = _cu(seqlens)
    x = wl.draw_block_scores(34, seqlens, hkv, kind="heavy")
    got = _gpu_select(x, cu, topk)
    tokens = np.unique(np.concatenate([np.random.default_rng(6).integers(0, T, 60), [0, 63, 64, 127, 128, T - 1]]))
    ref = tko.select_blocks(x, cu, topk, tokens=tokens)
    assert np.array_equal(got[tokens], ref[tokens])
    cur = (np.arange(T) // 64)[:, None, None]
    n_valid = np.minimum(cur + 1, topk)
    col = np.arange(topk)[None, None, :]
    assert np.array_equal(got >= 0, np.broadcast_to(col < n_valid, got.shape))
    assert (got <= cur).all()
    srt = np.sort(np.where(got < 0, -1 - col, got), axis=2)
    assert (np.diff(srt, axis=2) != 0).all()                      # no block twice in a row
    assert (got[:, :, 0] == 0).all()
    assert np.array_equal(got[64:, :, 1], np.broadcast_to(cur[64:, :, 0], (T - 64, hkv)))
    # free picks come in descending score order
    sc = np.take_along_axis(x, np.maximum(got, 0).astype(np.int64), axis=2)
    free = sc[4096:, :, 3:]
    assert (np.diff(free, axis=2) <= 0).all()


def test_selection_feeds_the_attention_path_on_the_device():
    """scores -> idx -> index inversion -> forward, all on the device, equals the oracle's forward on the oracle's idx."""
    print("case select then forward", flush=True)
    w = wl.realise(wl.small("g4"))
    cu = w.cu_seqlens
    x = wl.draw_block_scores(35, w.seqlens, w.hkv, kind="heavy")
    ref_idx = tko.select_blocks(x, cu, w.topk)
    cu_d = torch.from_numpy(cu).cuda()
    idx_d = nsa.select_blocks(torch.from_numpy(x).cuda(), cu_d, w.topk)
    attn = nsa.SelAttention(w.total_tokens, w.hq, w.hkv, w.topk, nseq=1, causal=True, bwd=False)
    from gpu_util import TOL_O, assert_close, dev_bf16, to_f64
    q, k, v = (dev_bf16(t) for t in (w.q, w.k, w.v))
    o, lse = attn.forward(q, k, v, idx_d, cu_d, rebuild_index=True)
    torch.cuda.synchronize()
    assert np.array_equal(idx_d.cpu().numpy(), ref_idx)
    Q, K, V = (wl.bf16_bits_to_f64(t) for t in (w.q, w.k, w.v))
    ro, _ = orc.forward(Q, K, V, ref_idx, cu, block=64, causal=True)
    assert_close("O", to_f64(o), ro, TOL_O)


def test_argument_errors():
    print("case select errors", flush=True)
    L = nsa.lib()
    x = torch.zeros(64, 1, 8, dtype=torch.float32, device="cuda")
    out = torch.empty(64, 1, 4, dtype=torch.int32, device="cuda")
    shape = nsa.Shape(64, 1, 1, 1, 128, 64, 4, 1, 0.0, 0)
    p = lambda t: C.c_void_p(t.data_ptr())
    assert L.nsa_sel_select_blocks(C.byref(shape), p(x), 8, None, 1, 2, None, None) == -1            # no output
    assert L.nsa_sel_select_blocks(C.byref(shape), None, 8, None, 1, 2, p(out), None) == 0            # no scores: forced blocks only
    torch.cuda.synchronize()
    assert out[63, 0].tolist() == [0, -1, -1, -1] and out[0, 0].tolist() == [0, -1, -1, -1]
    assert L.nsa_sel_select_blocks(C.byref(shape), p(x), 8, None, -1, 2, p(out), None) == -1
    assert L.nsa_sel_select_blocks(C.byref(shape), p(x), 0, None, 1, 2, p(out), None) == -2
    assert L.nsa_sel_select_blocks(C.byref(shape), p(x), 16385, None, 1, 2, p(out), None) == -2
    shape2 = nsa.Shape(64, 2, 1, 1, 128, 64, 4, 1, 0.0, 0)
    assert L.nsa_sel_select_blocks(C.byref(shape2), p(x), 8, None, 1, 2, p(out), None) == -1   # nseq > 1 needs cu
    shape3 = nsa.Shape(0, 1, 1, 1, 128, 64, 4, 1, 0.0, 0)
    assert L.nsa_sel_select_blocks(C.byref(shape3), p(x), 8, None, 1, 2, p(out), None) == 0     # nothing to do


@pytest.mark.parametrize("seqlens,hkv,topk,causal,kind,stride", [
    ([13000, 1, 107], 5, 16, True, "wild", None),
    ([13000, 107], 5, 16, True, "wild", 207),
    ([21846], 3, 32, False, "wild", None),
    ([70000], 1, 1, True, "ties", 1099),              # two chunks
    ([26000, 1, 214], 5, 16, True, "wild", None),     # 131075 rows: eight a wavefront, the last wavefront with three
    ([26000, 214], 5, 16, True, "wild", 407),         # 131070 rows: one a wavefront
    ([43691], 3, 32, False, "wild", None),            # a wavefront's rows begin and end inside a token
    ([70000], 2, 1, True, "ties", 1099),              # four tokens a wavefront, two chunks
    ([1000] * 524 + [289], 1, 16, True, "wild", 16),  # 524289 rows of one head: eight a wavefront, fewer lanes than the bound counts
    ([1000] * 524 + [287], 1, 16, True, "wild", 17),  # 524287: one
])
def test_rows_of_a_wavefront(seqlens, hkv, topk, causal, kind, stride):
    """From 131072 rows (524288 with one head) a wavefront takes eight, and scores are compared as floats: infinities, NaN, both zeros and
    denormals.  Oracle on sampled tokens."""
    print("case rows of a wavefront", seqlens, hkv, topk, causal, kind, stride, flush=True)
    cu, n = _cu(seqlens), sum(seqlens)
    x = wl.draw_block_scores(35, seqlens, hkv, kind=kind, stride=stride, trap_future=causal)
    tokens = np.unique(np.concatenate([np.random.default_rng(9).integers(0, n, 200), np.arange(n - 12, n), np.arange(12)]))
    ref = tko.select_blocks(x, cu, topk, causal=causal, tokens=tokens)
    got = _gpu_select(x, cu, topk, causal=causal)
    assert np.array_equal(got[tokens], ref[tokens])


def _narrow_scores(kind, rows, blocks, gen):
    z = torch.randn(rows, 1, blocks, generator=gen, device="cuda")
    if kind == "uniform":
        return torch.rand(rows, 1, blocks, generator=gen, device="cuda")
    if kind == "offset":
        return z + 10
    if kind == "flat":
        return torch.exp(0.1 * z) / blocks
    if kind == "mass":                              # attention mass of 64 keys with normal logits
        return sum(torch.randn(rows, 1, blocks, generator=gen, device="cuda").exp() for _ in range(64)) / (64 * blocks)
    if kind == "nan":
        return torch.where(torch.rand(rows, 1, blocks, generator=gen, device="cuda") < 0.3, float("nan"), z)
    return torch.exp(1.5 * z)


@pytest.mark.parametrize("kind", ["uniform", "offset", "flat", "mass", "nan"])
@pytest.mark.parametrize("topk", [16, 32])
def test_narrow_ranges_of_scores(kind, topk):
    """Scores of a narrow range, and rows with many NaNs: the picks against the oracle, and no more time than heavy-tailed scores take.
    Rows whose bound is too loose to rank their survivors go to the method of one pick a round, four to six times slower: such
    scores then took 1.4 (uniform, 16) to 6.3 times as long.  The fastest of several runs, with a margin for the chip of 1.3."""
    print("case narrow scores", kind, topk, flush=True)
    rows, blocks = 65536, 1024
    gen = torch.Generator(device="cuda").manual_seed(5)
    scores = {k: _narrow_scores(k, rows, blocks, gen) for k in (kind, "heavy")}
    pick = {k: (lambda x=x: nsa.select_blocks(x, None, topk, causal=False)) for k, x in scores.items()}
    tokens = np.random.default_rng(4).integers(0, rows, 40)
    x = scores[kind].cpu().numpy()
    ref = tko.select_blocks(x, np.array([0, rows], dtype=np.int32), topk, causal=False, tokens=tokens)
    assert np.array_equal(pick[kind]().cpu().numpy()[tokens], ref[tokens])
    fastest = dict.fromkeys(pick, float("inf"))
    start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    for _ in range(8):
        for k, run in pick.items():
            start.record()
            for _ in range(10):
                run()
            end.record()
            end.synchronize()
            fastest[k] = min(fastest[k], start.elapsed_time(end))
    assert fastest[kind] < 1.3 * fastest["heavy"], fastest


@pytest.mark.parametrize("blocks,kind", [(129, "heavy"), (132, "wild"), (136, "ties"), (137, "heavy"), (1140, "wild"), (1160, "ties")])
def test_partly_filled_chunks_keep_everything(blocks, kind):
    """Up to 136 scores of a chunk survive without a search at top-k 32, alone or after the survivors of a full chunk; what was not
    loaded (NaN beside -inf) never does."""
    print("case partly filled", blocks, kind, flush=True)
    rng, tokens, seqlens = np.random.default_rng(blocks), 60 if blocks < 1000 else 12, [blocks * 64 - 5]
    x = np.zeros((seqlens[0], 1, -(-blocks // 4) * 4), dtype=np.float32)        # only the first rows are looked at
    z = rng.standard_normal((tokens, 1, x.shape[2]))
    x[:tokens] = np.exp(1.5 * z) if kind == "heavy" else np.round(np.exp(1.5 * z)) if kind == "ties" else z
    if kind == "wild":
        x[:tokens][rng.random((tokens, 1, x.shape[2])) < 0.3] = np.nan
    x[:tokens:5, :, 3:] = -np.inf
    x[1:tokens:5, :, 40:] = np.nan
    got = _gpu_select(x, None, 32, causal=False)[:tokens]
    ref = tko.select_blocks(x, _cu(seqlens), 32, causal=False, tokens=range(tokens))
    assert np.array_equal(got, ref[:tokens])
