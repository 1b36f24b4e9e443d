"""The sizes at the edge of what the library accepts: the largest block count, thousands of packed sequences,
a call with no tokens at all."""
import numpy as np
import pytest
import torch

import paper_2508_18224_amd as nsa
import workloads as wl
from oracle import nsa_sel_oracle as orc
from gpu_util import BitsF64, Case, TOL_GRAD, TOL_O, TOL_LSE, assert_close, to_f64

pytestmark = pytest.mark.gpu


def _sampled(w, c, tokens):
    o, lse = c.forward()
    dq, dk, dv = c.backward(o, lse)
    Q, K, V, dO = (BitsF64(x) for x in (w.q, w.k, w.v, w.do))
    O_ref, LSE_ref = orc.forward(Q, K, V, w.idx, w.cu_seqlens, block=w.block, tokens=tokens)
    dQ_ref, _, _ = orc.backward(Q, K, V, dO, w.idx, w.cu_seqlens, block=w.block, tokens=tokens)
    sel = torch.tensor(tokens, device="cuda")
    assert_close("O", to_f64(o[sel]), O_ref[tokens], TOL_O)
    assert np.abs(to_f64(lse[sel]) - LSE_ref[tokens]).max() <= TOL_LSE
    assert_close("dQ", to_f64(dq[sel]), dQ_ref[tokens], TOL_GRAD)
    return dk, dv


def test_largest_block_count():
    """13 000 blocks of 64 tokens in one sequence, close to the limit the inversion's LDS tables set (one more
    thousand is refused): inversion bit-exact on whole lists, attention on sampled rows and one sampled KV block."""
    print("case block-count limit", flush=True)
    T = 13000 * 64
    assert nsa.lib().nsa_sel_workspace_bytes(nsa.Shape(14000 * 64, 1, 1, 1, 128, 64, 3, 1, 0.0, 0), None, None, None) == -2
    w = wl.realise(wl.Workload("limit", [T], hq=1, hkv=1, topk=3, sink=True, seed=81))
    c = Case(w)
    tokens = sorted({0, 63, 64, T - 1, *[int(x) for x in np.random.default_rng(1).integers(0, T, 10)]})
    dk, dv = _sampled(w, c, tokens)
    cnt, off, qlist, qslot, vmask, bcap = c.attn.index_arrays()
    rc, ro, rl, rs, rv = orc.invert_index(w.idx, w.cu_seqlens)
    assert np.array_equal(cnt[:, :rc.shape[1]], rc) and np.array_equal(qlist, rl) and np.array_equal(qslot, rs)
    Q, K, V, dO = (BitsF64(x) for x in (w.q, w.k, w.v, w.do))
    (dKb, dVb), = orc.backward_kv_blocks(Q, K, V, dO, w.idx, w.cu_seqlens, [(0, 0, 12999)])
    assert_close("dK last block", to_f64(dk[12999 * 64:, 0]), dKb, TOL_GRAD)
    assert_close("dV last block", to_f64(dv[12999 * 64:, 0]), dVb, TOL_GRAD)


def test_thousands_of_packed_sequences():
    """2 500 sequences of 1 .. 130 tokens (most shorter than a block, some empty): every sequence owns its blocks."""
    print("case many sequences", flush=True)
    rng = np.random.default_rng(82)
    seqlens = [int(x) for x in rng.integers(0, 131, 2500)]
    w = wl.realise(wl.Workload("many", seqlens, hq=4, hkv=2, topk=4, seed=82))
    T = w.total_tokens
    c = Case(w)
    tokens = sorted({0, T - 1, *[int(x) for x in rng.integers(0, T, 300)]})
    _sampled(w, c, tokens)
    cnt, off, qlist, qslot, vmask, bcap = c.attn.index_arrays()
    rc, ro, rl, rs, rv = orc.invert_index(w.idx, w.cu_seqlens)
    assert np.array_equal(cnt[:, :rc.shape[1]], rc) and np.array_equal(qlist, rl) and np.array_equal(vmask, rv)


def test_no_tokens_at_all():
    print("case zero tokens", flush=True)
    attn = nsa.SelAttention(0, 4, 2, 8, nseq=1)
    import ctypes as C
    L = nsa.lib()
    assert attn.fwd_ws.numel() == 0                       # a zero-byte workspace has no address
    rc = L.nsa_sel_build_index(C.byref(attn.shape), None, None, None, 0, None)
    assert rc == 0
    rc = L.nsa_sel_fwd(C.byref(attn.shape), None, None, None, None, None, 1, None, 0, None, None, None, 0, None)
    assert rc == 0
    rc = L.nsa_sel_bwd(C.byref(attn.shape), None, None, None, None, None, None, None, None, 0, None, None, None, None,
                       0, None)
    assert rc == 0
    torch.cuda.synchronize()


@pytest.mark.parametrize("singles,dense", [(0, True), (0, False), (0, None), (40, True), (40, False)])
def test_tokens_past_the_last_sequence(singles, dense):
    """A padded batch, cu_seqlens ending before total_tokens: the tokens past it are queries of the last sequence, and every
    row of the result is written.  With the keys of the padding never selected that is what the oracle gives for a last
    sequence that reaches to the end; 40 one-token sequences in front take the inversion's walk by token, and without them the library's
    choice is the short forward, which finds its tiles and rows by itself."""
    print("case padded batch", singles, dense, flush=True)
    seqlens = [1] * singles + [130, 192 + 178]                     # the last sequence: 192 tokens and 178 of padding
    w = wl.realise(wl.Workload("padded", seqlens, hq=4, hkv=2, topk=6, sink=True, seed=84))
    T, end = w.total_tokens, w.total_tokens - 178
    last = w.idx[end - 192:]
    last[last >= 3] = -1                                           # the padding's own blocks
    c = Case(w, dense=dense)
    c.cu[-1] = end
    o, lse = c.forward()
    dq, dk, dv = c.backward(o, lse)
    Q, K, V, dO = c.host_f64()
    rO, rL = orc.forward(Q, K, V, w.idx, w.cu_seqlens)
    rq, rk, rv = orc.backward(Q, K, V, dO, w.idx, w.cu_seqlens)
    assert_close("O", to_f64(o), rO, TOL_O)
    assert np.abs(to_f64(lse) - rL)[np.isfinite(rL)].max() <= TOL_LSE
    assert_close("dQ", to_f64(dq), rq, TOL_GRAD)
    assert_close("dK", to_f64(dk[:end]), rk[:end], TOL_GRAD)
    assert_close("dV", to_f64(dv[:end]), rv[:end], TOL_GRAD)


@pytest.mark.parametrize("block,window", [(64, 0), (64, 512), (128, 0), (128, 512)])
def test_query_tensors_beyond_4_gb(block, window):
    """Q, O, dO and dQ of 4.6 GB, whose rows 32-bit offsets do not reach (64 heads, 280 000 tokens in two sequences): every
    output is that of the two sequences taken alone, 2.3 GB each, bit for bit - same lists, same work units."""
    print("case beyond 4 GB", block, window, flush=True)
    hq, hkv, lengths = 64, 8, [139000, 141000]
    T, cuts = sum(lengths), [0, lengths[0], sum(lengths)]
    gen = torch.Generator(device="cuda").manual_seed(85)

    def normal(heads):
        return torch.randn(T, heads, 128, generator=gen, device="cuda", dtype=torch.float32).to(torch.bfloat16)
    q, k, v, do = normal(hq), normal(hkv), normal(hkv), normal(hq)
    cu = torch.tensor(cuts, dtype=torch.int32, device="cuda")
    if window:
        idx = nsa.window_blocks(T, hkv, window, cu, block=block)
    else:  # own block, sink, and one earlier block
        own = torch.cat([torch.arange(n, device="cuda") // block for n in lengths])[:, None]
        pick = (torch.rand(T, hkv, generator=gen, device="cuda") * own).long()
        idx = torch.stack([own.expand(T, hkv), torch.zeros_like(pick), pick], dim=2).to(torch.int32).contiguous()

    def step(a, b, cu):
        attn = nsa.SelAttention(b - a, hq, hkv, idx.shape[2], nseq=1 if cu is None else 2, block=block, window=window,
                                unit=2048, dense=True, ws_cap_bytes=1)
        o, lse = attn.forward(q[a:b], k[a:b], v[a:b], idx[a:b], cu)
        return (o, lse, *attn.backward(q[a:b], k[a:b], v[a:b], o, lse, do[a:b], cu))
    whole = step(0, T, cu)
    for a, b in zip(cuts, cuts[1:]):
        for nm, x, y in zip(("O", "LSE", "dQ", "dK", "dV"), step(a, b, None), whole):
            assert torch.equal(x, y[a:b]), nm
    assert bool(torch.isfinite(whole[0][::997].float()).all())
