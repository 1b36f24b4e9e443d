"""The order in which the main kernels take the work units.  The backward's draw their work units from a counter where there are some thousands of them (see UnitQueue in
csrc/bwd.hip).  Which workgroup computes a unit changes nothing about it: the results are those of a workgroup a unit, which
small enough a workspace brings about (few KV heads a pass, few units), bit for bit, and the same every time.
The forward's take the KV heads in turn or one after the other (units_in_turn in csrc/common.h), with the same results."""
import pytest
import torch

import paper_2508_18224_amd as nsa
import workloads as wl
from gpu_util import Case

pytestmark = pytest.mark.gpu
MIN_UNITS = 2048  # of the rule


def _bound(w, hkv, unit):
    blocks = w.total_tokens // w.block + len(w.seqlens)
    return hkv * blocks + hkv * w.total_tokens * w.topk // unit + 1


#        lengths, query heads, KV heads, top-k, block, window, units at most, KV heads a pass (0: all)
CASES = [([4096], 8, 8, 16, 64, 0, 2569, 0),                     # all lists ordered
         ([2000, 1, 64, 1500, 531], 16, 8, 16, 64, 0, 2601, 0),  # packed, ragged, g = 2
         ([12000], 40, 8, 8, 64, 0, 4505, 0),                    # more than half a unit for each slot, g = 5
         ([5000], 8, 8, 9, 64, 512, 2039, 0),                # below the rule's least: a workgroup a unit
         ([8192], 8, 8, 9, 64, 512, 3337, 0),                    # the window's form
         ([4096], 16, 8, 16, 128, 0, 2313, 0),                   # 128-token blocks
         ([8192], 8, 8, 5, 128, 512, 1801, 0),                   # their window, below the least
         ([16384], 16, 16, 5, 128, 512, 7185, 0),                # and above
         ([4096], 20, 20, 16, 64, 0, 6421, 11),                  # two passes, a counter each, by number
         ([16384], 16, 16, 16, 128, 0, 18449, 0)]                # more units than the order has room for: by number


@pytest.mark.parametrize("lengths,hq,hkv,topk,block,window,units,heads", CASES)
def test_units_from_the_queue_are_those_of_a_workgroup_each(lengths, hq, hkv, topk, block, window, units, heads):
    w = wl.realise(wl.Workload("queue", lengths, hq=hq, hkv=hkv, topk=topk, sink=True, seed=3, block=block))
    assert _bound(w, hkv, 256) == units
    case = Case(w, window=window)

    def attention(cap=None):
        return nsa.SelAttention(w.total_tokens, hq, hkv, topk, nseq=len(lengths), block=block, window=window, unit=256, ws_cap_bytes=cap)
    idx = case.idx
    if window:
        idx = nsa.window_blocks(w.total_tokens, hkv, window, case.cu, block=block)
        assert idx.shape[2] == topk
    whole = attention()
    if heads:  # a workspace of `heads` KV heads: more than the least number of units a pass
        rows = lambda n: w.total_tokens * n * (hq // hkv) * topk * 256 + _bound(w, n, 256) * 2 * block * 512
        whole = attention(rows(heads) + w.total_tokens * hq * 8 + 1024)
        assert whole.bwd_ws.numel() < nsa.workspace_bytes(whole.shape)[1] and _bound(w, heads, 256) >= MIN_UNITS
    single = attention(0)  # one KV head a pass
    assert _bound(w, 1, 256) < MIN_UNITS
    o, lse = whole.forward(case.q, case.k, case.v, idx, case.cu)
    single.build_index(idx, case.cu)
    single.bwd_ws.fill_(0x7F)
    want = single.backward(case.q, case.k, case.v, o, lse, case.do, case.cu)
    assert all(bool(torch.isfinite(x).all()) for x in want)
    for _ in range(3):
        whole.bwd_ws.fill_(0x7F)  # counters and order are made anew by every call
        got = whole.backward(case.q, case.k, case.v, o, lse, case.do, case.cu)
        for name, a, b in zip(("dQ", "dK", "dV"), got, want):
            assert torch.equal(a.view(torch.int16), b.view(torch.int16)), name


def _queue(attn, w, lengths, block):
    """(counters, order) the last backward left in the room of the last unit's sums; None where it had no queue (and 0x7F was filled in)."""
    room = attn.bwd_ws[-2 * block * 512:].view(torch.int32).cpu().numpy()
    return None if (room[:64] == 0x7F7F7F7F).all() else (room[:64], room[64:])


@pytest.mark.parametrize("lengths,hq,hkv,topk,block,causal,queued", [
    ([4096], 8, 8, 16, 64, True, True), ([2000, 1, 64, 1500, 531], 16, 8, 16, 64, True, True), ([4096], 16, 8, 16, 128, True, True),
    ([12000], 40, 8, 8, 64, True, True), ([12000], 32, 8, 8, 64, True, False),  # more than half a unit for each slot, g = 5 and 4
    ([8192], 8, 8, 8, 64, False, True),      # lists of about two units of 256
    ([8192], 8, 8, 2, 64, False, False),     # of half a unit: all alike and one unit each
    ([8192], 8, 8, 2, 64, True, False)])     # (too few units)
def test_order_of_the_units(lengths, hq, hkv, topk, block, causal, queued):
    """Long units first, in classes that part where lists of like length don't, each class by number."""
    w = wl.realise(wl.Workload("order", lengths, hq=hq, hkv=hkv, topk=topk, sink=causal, seed=4, block=block, causal=causal))
    case = Case(w)
    attn = nsa.SelAttention(w.total_tokens, hq, hkv, topk, nseq=len(lengths), block=block, unit=256, causal=causal)
    o, lse = attn.forward(case.q, case.k, case.v, case.idx, case.cu)
    attn.bwd_ws.fill_(0x7F)
    attn.backward(case.q, case.k, case.v, o, lse, case.do, case.cu)
    found = _queue(attn, w, lengths, block)
    assert (found is not None) == queued
    if not queued:
        return
    cnt = attn.index_arrays()[0].ravel()
    units = [min(256, n - at) for n in map(int, cnt) for at in range(0, n, 256)]
    slots = 512 if block == 64 else 256
    assert found[0][0] == len(units) or found[0][0] >= len(units) - slots  # every workgroup drew until nothing was left
    want = sorted(range(len(units)), key=lambda u: (units[u] * 8 <= 3 * 256) + (units[u] * 16 <= 3 * 256))
    assert list(found[1][:len(units)]) == want


def test_all_keys_by_number():
    """32768 tokens, 32 heads, all keys: lists of half a unit, which the length classes once split down the middle."""
    w = wl.Workload("like", [32768], hq=32, hkv=8, topk=16, causal=False)
    attn = nsa.SelAttention(32768, 32, 8, 16, causal=False)
    gen = torch.Generator(device="cuda").manual_seed(3)
    q, do = (torch.randn(32768, 32, 128, generator=gen, device="cuda").bfloat16() for _ in range(2))
    k, v = (torch.randn(32768, 8, 128, generator=gen, device="cuda").bfloat16() for _ in range(2))
    idx = torch.rand(32768, 8, 512, generator=gen, device="cuda").argsort(dim=2)[..., :16].int().contiguous()
    o, lse = attn.forward(q, k, v, idx)
    attn.bwd_ws.fill_(0x7F)
    attn.backward(q, k, v, o, lse, do)
    assert _queue(attn, w, [32768], 64) is None


def test_heads_in_turn_where_their_number_suits():
    """A number of KV heads that is no multiple of eight costs the forward's main kernel no more a head than one that is (in turn the XCDs
    would gather from the Q of all of them: 1.3 times as long)."""
    times = {}
    for heads in (21, 24):
        T, topk = 7407, 32
        gen = torch.Generator(device="cuda").manual_seed(6)
        q, k, v = (torch.randn(T, heads, 128, generator=gen, device="cuda").bfloat16() for _ in range(3))
        idx = torch.rand(T, heads, 116, generator=gen, device="cuda").argsort(dim=2)[..., :topk].int().contiguous()
        attn = nsa.SelAttention(T, heads, heads, topk, causal=False, bwd=False)
        best = float("inf")
        for rep in range(8):
            nsa.binding.profile_enable(64)
            attn.forward(q, k, v, idx)
            torch.cuda.synchronize()
            best = min(best, nsa.binding.profile_collect()["fwd_main"][0])
            nsa.binding.profile_enable(0)
        times[heads] = best / heads
    assert times[21] < 1.15 * times[24], times


@pytest.mark.parametrize("lengths,g,hkv,block,part", [([8200], 1, 40, 64, 8), ([16385], 4, 8, 64, 4), ([9000, 1, 7400], 2, 16, 128, 4)])
def test_forward_of_all_heads_and_of_a_few_agree(lengths, g, hkv, block, part):
    T, topk = sum(lengths), 8
    most = 1 << (18 if g == 1 else 19)  # (of units_in_turn; the parts are of a number of heads that it takes in turn)
    assert part * g * T <= most < hkv * g * T  # the few in turn, all of them head by head
    gen = torch.Generator(device="cuda").manual_seed(5)
    q = torch.randn(T, hkv * g, 128, generator=gen, device="cuda").to(torch.bfloat16)
    k, v = (torch.randn(T, hkv, 128, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2))
    cu = torch.tensor([sum(lengths[:i]) for i in range(len(lengths) + 1)], dtype=torch.int32, device="cuda")
    stride = -(-max(lengths) // block)
    idx = nsa.select_blocks(torch.rand(T, hkv, stride + -stride % 4, generator=gen, device="cuda"), cu, topk, block=block)

    def forward(j0, n):
        attn = nsa.SelAttention(T, n * g, n, topk, nseq=len(lengths), block=block, unit=512, dense=g > 1, bwd=False)
        kv = slice(j0, j0 + n)
        return attn.forward(q[:, j0 * g:(j0 + n) * g].contiguous(), k[:, kv].contiguous(), v[:, kv].contiguous(),
                            idx[:, kv].contiguous(), cu)
    o, lse = forward(0, hkv)
    assert bool(torch.isfinite(lse).all())
    for j0 in range(0, hkv, part):
        n = min(part, hkv - j0)
        o_part, lse_part = forward(j0, n)
        assert torch.equal(o[:, j0 * g:(j0 + n) * g].view(torch.int16), o_part.view(torch.int16)), j0
        assert torch.equal(lse[:, j0 * g:(j0 + n) * g].view(torch.int32), lse_part.view(torch.int32)), j0
