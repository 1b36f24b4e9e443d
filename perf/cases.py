"""What this library is timed on: passes through its public entry points, from the smallest call to the largest.

A case is a dict of plain values:
  op       "train"   forward + backward through torch.autograd (selected_attention): O, LSE, dQ, dK, dV
           "gated"   the same with the gate of the branch combination: O_out, dQ, dK, dV, dgate
           "window"  the sliding-window branch, forward + backward (`window` tokens)
           "prefill" forward alone with a caller-owned workspace (SelAttention.forward)
           "static"  forward alone that allocates no workspace (SelAttention.forward_static)
           "select"  block scores -> selection tensor (select_blocks), the step in front of the attention
  lengths  sequence lengths, comma separated (several: a packed batch)
  hq, hkv, topk, block, causal
  sink, recent, local   the selection: block 0 forced, this many most recent blocks forced (the own one is always
           among them), this many picks from the 8 blocks before those; the rest uniform over earlier blocks
           (over all blocks when not causal)

Every forward includes the inversion of the selection tensor: a model draws a new selection in every layer and step.
"""
from __future__ import annotations

import math

import torch

import paper_2508_18224_amd as nsa

HEAD_DIM = 128
LOCAL_WINDOW = 8
DEVICE = "cuda:0"
TRAINING = ("train", "gated", "window")


def _case(name, op, lengths, hq, hkv, topk, block=64, causal=True, sink=True, recent=1, local=0, window=0):
    case = dict(op=op, lengths=",".join(str(n) for n in lengths), hq=hq, hkv=hkv, topk=topk, block=block,
                causal=causal, sink=sink, recent=recent, local=local, window=window)
    return dict(name=name, **case) if name else case


def listed():
    return [
        # a unit-test sized training step: launches and host time
        _case("train_1k_g4", "train", [1024], 4, 1, 8, sink=False),
        # a serving loop that may not allocate: prompt of a few hundred words, 8 heads of a sharded model
        _case("static_2k_g4", "static", [2000], 8, 2, 16),
        # fine-tuning on a packed batch of short documents without causal mask
        _case("train_docs_bidir_g2", "train", [700, 64, 1, 333, 1029, 2300, 450], 8, 4, 8, causal=False, sink=False),
        # the lower end of the paper's grid, one KV head per query head
        _case("train_8k_g1", "train", [8192], 32, 32, 16),
        # a Llama-3-8B-shaped layer with the branch gate fused
        _case("gated_32k_g4", "gated", [32768], 32, 8, 16),
        # the sliding-window branch of the same layer
        _case("window_32k_g4", "window", [32768], 32, 8, 9, window=512),
        # packed long documents of uneven length, no head sharing
        _case("train_varlen_g1", "train", [23456, 4100, 17031, 9999, 31744, 5003, 12289, 6145], 16, 16, 16, sink=False),
        # Qwen-shaped heads, half of the free picks near the token
        _case("train_64k_g7_local", "train", [65536], 28, 4, 16, local=7),
        # the benchmark's shape, with 64-token and with 128-token blocks
        _case("train_64k_g4", "train", [65536], 32, 8, 16),
        _case("train_64k_g4_b128", "train", [65536], 32, 8, 8, block=128),
        # prefill of a 128K prompt, Llama-3-70B-shaped heads
        _case("prefill_128k_g8", "prefill", [131072], 64, 8, 16, recent=2),
        # choosing the blocks of a 64K prompt from their scores
        _case("select_64k", "select", [65536], 8, 8, 16, recent=2),
    ]


# No drawn case has more (token, head, selected key) products, forward and backward together, than the largest listed
# one: the backward counts 2.5 forwards.
_MOST_PRODUCTS = 3.5 * 65536 * 32 * 16 * 64


def draw(rng):
    """One more case of the ranges above (rng: random.Random)."""
    while True:
        op = rng.choices(["train", "gated", "window", "prefill", "static", "select"], [10, 3, 3, 3, 2, 2])[0]
        block = rng.choice([64, 64, 128])
        hkv = rng.choice([1, 2, 4, 5, 8, 16])
        g = rng.choice([1, 2, 4, 4, 5, 7, 8])
        most = {"static": 4000, "prefill": 131072}.get(op, 65536)
        tokens = int(round(math.exp(rng.uniform(math.log(1000), math.log(most)))))
        if rng.random() < 0.4:
            tokens = max(1024, tokens // 1024 * 1024)
        lengths = [tokens]
        if rng.random() < 0.35 and op != "select":
            cuts = sorted(rng.sample(range(1, tokens), rng.randint(1, 9)))
            lengths = [b - a for a, b in zip([0] + cuts, cuts + [tokens])]
        window, causal = 0, rng.random() < 0.85 or op in ("window", "select")
        topk = rng.choice([4, 8, 8]) if block == 128 else rng.choice([8, 16, 16, 16, 32])
        if op == "window":
            window = rng.choice([100, 256, 512, 512, 1000])
            topk = -(-(window - 1) // block) + 1
        sink = causal and rng.random() < 0.7
        recent = rng.choice([1, 1, 2])
        local = rng.choice([0, 0, (topk - 2) // 2])
        products = (3.5 if op in TRAINING else 1.0) * tokens * hkv * g * topk * block
        scratch = tokens * g * topk * 260 + 1024  # of one KV head; what forward_static holds is 64 MiB
        if products > _MOST_PRODUCTS or (op == "static" and scratch > 64 << 20):
            continue
        if op == "select" and tokens * hkv * (tokens // block + 4) * 4 > 2.2e9:
            continue
        return _case(None, op, lengths, hkv if op == "select" else hkv * g, hkv, topk, block, causal, sink,
                     recent, local if causal else 0, window)


def _lengths(case):
    return [int(n) for n in case["lengths"].split(",")]


def _pick(gen, count, m):
    """m distinct uniform integers of [0, count[row]) per row (Floyd's algorithm), -1 where there are fewer."""
    take = count.clamp(max=m)
    out = torch.full((count.numel(), m), -1, dtype=torch.int64, device=DEVICE)
    for i in range(m):
        top = count - take + i
        x = (torch.rand(count.numel(), generator=gen, dtype=torch.float64, device=DEVICE) * (top + 1)).long()
        x = torch.minimum(x, top)
        x = torch.where((out[:, :i] == x[:, None]).any(dim=1), top, x)
        out[:, i] = torch.where(i < take, x, -1)
    return out


def _selection(case, gen):
    """int32 [tokens, hkv, topk]: forced blocks, then the picks, then -1."""
    block, topk, hkv, sink, recent = case["block"], case["topk"], case["hkv"], case["sink"], case["recent"]
    rows = []
    for n in _lengths(case):
        own = (torch.arange(n, device=DEVICE) // block).repeat_interleave(hkv)
        if not case["causal"]:
            x = _pick(gen, torch.full_like(own, -(-n // block) - 1), topk - 1)
            cols = torch.cat([own[:, None], torch.where(x >= own[:, None], x + 1, x)], dim=1)
        else:
            forced = [torch.zeros_like(own)] if sink else []
            lo = 1 if sink else 0
            forced += [torch.where(own - r >= lo, own - r, -1) for r in range(recent)]
            hi = (own - recent + 1).clamp(min=lo)
            near = (hi - LOCAL_WINDOW).clamp(min=lo) if case["local"] else hi
            free = topk - len(forced)
            parts = [torch.stack(forced, dim=1)]
            for start, end, m in ((near, hi, case["local"]), (torch.full_like(hi, lo), near, free - case["local"])):
                if m > 0:
                    x = _pick(gen, end - start, m)
                    parts.append(torch.where(x >= 0, x + start[:, None], -1))
            cols = torch.cat(parts, dim=1)
            cols = cols.gather(1, torch.argsort((cols < 0).to(torch.int8), dim=1, stable=True))
        rows.append(cols.view(n, hkv, topk))
    return torch.cat(rows).to(torch.int32).contiguous()


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    lengths, op = _lengths(case), case["op"]
    tokens, hq, hkv = sum(lengths), case["hq"], case["hkv"]
    cu = None
    if len(lengths) > 1:
        cu = torch.tensor([sum(lengths[:i]) for i in range(len(lengths) + 1)], dtype=torch.int32, device=DEVICE)
    if op == "select":
        # attention mass per block: positive, heavy-tailed, more of it on recent blocks
        blocks = -(-(-(-max(lengths) // case["block"])) // 4) * 4
        scores = torch.randn(tokens, hkv, blocks, generator=gen, device=DEVICE).mul_(1.5).exp_()
        age = torch.arange(tokens, device=DEVICE)[:, None] // case["block"] - torch.arange(blocks, device=DEVICE)
        scores *= (1 + 2 * torch.exp(-age.clamp(min=0) / 8.0))[:, None, :]
        return dict(case=case, scores=scores, cu=cu)

    def normal(heads):
        return torch.randn(tokens, heads, HEAD_DIM, generator=gen, device=DEVICE).to(torch.bfloat16)

    state = dict(case=case, cu=cu, q=normal(hq), k=normal(hkv), v=normal(hkv))
    if op == "window":
        state["idx"] = nsa.window_blocks(tokens, hkv, case["window"], cu, block=case["block"], device=DEVICE)
    else:
        state["idx"] = _selection(case, gen)
    wrt = [state["q"], state["k"], state["v"]]
    if op in TRAINING:
        state["do"] = normal(hq)
    if op == "gated":
        state["gate"] = torch.sigmoid(1.5 * torch.randn(tokens, hq, generator=gen, device=DEVICE))
        state["others"] = normal(hq)
        wrt.append(state["gate"])
    if op in TRAINING:
        for x in wrt:
            x.requires_grad_(True)
    state["wrt"] = wrt
    state["attn"] = nsa.SelAttention(tokens, hq, hkv, case["topk"], nseq=len(lengths), causal=case["causal"],
                                     block=case["block"], window=case["window"], bwd=op in TRAINING, device=DEVICE)
    return state


def run(state):
    case, cu = state["case"], state["cu"]
    op = case["op"]
    if op == "select":
        return nsa.select_blocks(state["scores"], cu, case["topk"], block=case["block"], causal=case["causal"],
                                 n_sink=int(case["sink"]), n_local=case["recent"])
    q, k, v, idx, attn = state["q"], state["k"], state["v"], state["idx"], state["attn"]
    if op == "prefill":
        return attn.forward(q, k, v, idx, cu)
    if op == "static":
        return attn.forward_static(q, k, v, idx, cu)
    if op == "gated":
        out = nsa.selected_attention(q, k, v, idx, attn, cu, gate=state["gate"], o_acc=state["others"])
        return (out.detach(), *torch.autograd.grad(out, state["wrt"], state["do"]))
    out, lse = nsa.selected_attention(q, k, v, idx, attn, cu)
    return (out.detach(), lse.detach(), *torch.autograd.grad(out, state["wrt"], state["do"]))


def _kept_pairs(case):
    """(token, visible selected key) pairs of one query head: a block counts up to the token and inside the window."""
    total = 0
    for n in _lengths(case):
        if case["window"]:
            w = case["window"]
            total += n * w - w * (w - 1) // 2 if n >= w else n * (n + 1) // 2
            continue
        block = case["block"]
        nb = -(-n // block)
        if not case["causal"]:
            total += n * min(case["topk"] * block, n)
            continue
        for b in range(nb):
            rows = min(block, n - b * block)
            total += rows * min(case["topk"] - 1, b) * block + rows * (rows + 1) // 2
    return total


def work(case):
    lengths = _lengths(case)
    tokens, hq, hkv, op = sum(lengths), case["hq"], case["hkv"], case["op"]
    if op == "select":
        visible = sum(min(t // case["block"] + 1, -(-n // case["block"])) for n in lengths for t in range(n))
        return {"bytes": 4 * hkv * (visible + tokens * case["topk"]), "flops": 0}
    row_q, row_kv = 2 * HEAD_DIM * hq, 2 * HEAD_DIM * hkv
    fwd = tokens * (2 * row_q + 2 * row_kv + 4 * hq + 4 * hkv * case["topk"])
    bwd = tokens * (4 * row_q + 4 * row_kv + 4 * hq) if op in TRAINING else 0
    if op == "gated":
        fwd += tokens * (2 * row_q + 4 * hq)
        bwd += tokens * 8 * hq
    flops = 4 * HEAD_DIM * hq * _kept_pairs(case)
    return {"bytes": fwd + bwd, "flops": int(flops * (3.5 if op in TRAINING else 1.0))}


def tolerance(case):
    if case["op"] == "select":
        return "exact"
    return {"rel": 1e-2}
