"""Timed cases of the library's public entry points: the collectives a user's program calls, over the sizes,
rank counts, dtypes and options they are called with.

A case is a dict of plain values.  `prepare` builds on the GPU what a program has in hand before the call
(rank buffers, routing tables, an uploaded layout, a Prepared call), `run` makes one pass through the
tensor API of `paper_2608_00867_amd.nuna`, and `exact` computes the same outputs in float64 with torch alone.

All reductions add the ranks in ascending order in fp32 and round once, and all other calls move bytes: the
library promises the same bits whatever the placement, algorithm or launch shape, so every tolerance is
"exact".
"""
import math

import torch

from paper_2608_00867_amd import nuna

HIDDEN_DENSE = 8192  # token rows of the dense decode and prefill all-reduces
HIDDEN_MOE = 7168    # token rows of the MoE layer
EXPERTS = 256
TOPK = 8

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
ESIZE = {"bf16": 2, "f32": 4}
MIB = 1 << 20


def listed():
    return [
        # One decode step's tensor-parallel all-reduce, 4 tokens: the smallest call, bound by latency.  A
        # serving loop repeats it on the same buffers, so it keeps the Prepared call.
        dict(name="ar_decode", op="allreduce", ranks=8, dtype="bf16", count=4 * HIDDEN_DENSE, prepared=True),
        # The same over a 64-rank domain: many short streams per element.
        dict(name="ar_ranks64", op="allreduce", ranks=64, dtype="bf16", count=128 * 1024, prepared=True),
        # A rank count that is no power of two (half of a 24-GPU group), a short prefill of 512 tokens.
        dict(name="ar_ranks12", op="allreduce", ranks=12, dtype="bf16", count=512 * HIDDEN_DENSE, prepared=False),
        # A gradient bucket of about 25 MiB in fp32, of an odd number of elements.
        dict(name="ar_grad_ragged", op="allreduce", ranks=8, dtype="f32", count=6553603, prepared=False),
        # Prefill of 4096 tokens, the largest activation all-reduce.
        dict(name="ar_prefill", op="allreduce", ranks=8, dtype="bf16", count=4096 * HIDDEN_DENSE, prepared=False),
        # Sharded gradients: reduce-scatter in fp32, 4 MiB shards.
        dict(name="rs_f32", op="reduce_scatter", ranks=8, dtype="f32", count=MIB),
        # Sharded weights: all-gather of 1 MiB shards over 16 ranks.
        dict(name="ag_ranks16", op="all_gather", ranks=16, dtype="bf16", count=MIB // 2),
        # A flat weight buffer cut into equal shards that are no whole number of 16-byte vectors.
        dict(name="ag_ragged", op="all_gather", ranks=8, dtype="bf16", count=1048583),
        # MoE prefill: the dispatch of 512 tokens a rank with a layout the program keeps.
        dict(name="moe_dispatch", op="dispatch", ranks=8, dtype="bf16", tokens=512, hidden=HIDDEN_MOE, topk=TOPK,
             experts=EXPERTS),
        # The way back, gate-weighted.
        dict(name="moe_combine", op="combine", ranks=8, dtype="bf16", tokens=512, hidden=HIDDEN_MOE, topk=TOPK,
             experts=EXPERTS, weighted=True),
        # A larger decode batch whose routing is read where the gate kernel left it.
        dict(name="moe_routed", op="routed", ranks=8, dtype="bf16", tokens=128, hidden=HIDDEN_MOE, topk=TOPK,
             experts=EXPERTS),
        # One serving step with a new routing: plan it, upload it, dispatch, combine, free the layout.
        dict(name="moe_step", op="step", ranks=8, dtype="bf16", tokens=128, hidden=HIDDEN_MOE, topk=TOPK,
             experts=EXPERTS),
    ]


def _log_uniform(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def _count(rng, dtype, least, most):
    """Elements for a buffer of least..most bytes: half of them whole 16-byte vectors (rows of a model's
    width), the others any number."""
    n = max(1, _log_uniform(rng, least, most) // ESIZE[dtype])
    if rng.random() < 0.5:
        n = max(64, n // 64 * 64)
    return n


def draw(rng):
    op = rng.choice(["allreduce"] * 4 + ["reduce_scatter"] * 2 + ["all_gather"] * 2 +
                    ["dispatch", "combine", "routed", "step"])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    if op == "allreduce":
        ranks = rng.choice([2, 3, 4, 6, 8, 8, 8, 12, 16, 24, 32, 64])
        # At most 256 MiB of inputs, 48 MiB a rank.
        count = _count(rng, dtype, 16 << 10, min(48 * MIB, 256 * MIB // ranks))
        return dict(op=op, ranks=ranks, dtype=dtype, count=count, prepared=rng.random() < 0.5)
    if op in ("reduce_scatter", "all_gather"):
        ranks = rng.choice([2, 3, 4, 6, 8, 8, 8, 12, 16, 32])
        # At most 192 MiB on the side that holds a shard per rank and rank, 16 MiB a shard.
        count = _count(rng, dtype, 4 << 10, min(16 * MIB, 192 * MIB // ranks ** 2))
        return dict(op=op, ranks=ranks, dtype=dtype, count=count)
    ranks = rng.choice([4, 8, 8, 16])
    experts = ranks * rng.choice([1, 4, 8, 32])
    c = dict(op=op, ranks=ranks, dtype=dtype, tokens=_log_uniform(rng, 1, (128 if op == "step" else 512) * 8 // ranks),
             hidden=rng.choice([2048, 2880, 4096, 5120, 7168]), topk=min(experts, rng.choice([1, 2, 4, 6, 8])),
             experts=experts)
    if op == "combine":
        c["weighted"] = rng.random() < 0.5
    return c


def _values(n, dtype, gen):
    return torch.randn(n, generator=gen, device="cuda").to(DTYPES[dtype])


def _routing(case, gen):
    """int32 [P, T, k]: k distinct experts of each token, uniform."""
    keys = torch.rand((case["ranks"], case["tokens"], case["experts"]), generator=gen, device="cuda")
    return keys.topk(case["topk"], dim=2).indices.to(torch.int32).contiguous()


def _inputs(case, seed):
    """What both sides start from: rank buffers, or the routing table, token rows and gate weights."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    P, dtype = case["ranks"], case["dtype"]
    if case["op"] in ("allreduce", "reduce_scatter", "all_gather"):
        n = case["count"] * (P if case["op"] == "reduce_scatter" else 1)
        return {"in": [_values(n, dtype, gen) for _ in range(P)]}
    T, H = case["tokens"], case["hidden"]
    s = {"topk": _routing(case, gen)}
    if case["op"] == "combine":
        rows = [int(v) for v in _sent(case, s["topk"]).sum(dim=0)]
        s["y"] = [_values(max(rows) * H, dtype, gen).view(max(rows), H) for _ in range(P)]
        s["weights"] = torch.rand((P, T, P), generator=gen, device="cuda") if case["weighted"] else None
    else:
        s["send"] = [_values(T * H, dtype, gen).view(T, H) for _ in range(P)]
    return s


def prepare(case, seed):
    nuna.init()
    s = _inputs(case, seed)
    s["case"] = case
    op, P, dtype = case["op"], case["ranks"], DTYPES[case["dtype"]]

    def buffers(*shape):
        return [torch.zeros(shape, dtype=dtype, device="cuda") for _ in range(P)]

    if op == "allreduce":
        s["out"] = buffers(case["count"])
        if case["prepared"]:
            s["call"] = nuna.prepare_allreduce(s["in"], s["out"])
    elif op == "reduce_scatter":
        s["out"] = buffers(case["count"])
    elif op == "all_gather":
        s["out"] = buffers(P * case["count"])
    else:
        T, H, E = case["tokens"], case["hidden"], case["experts"]
        if op in ("dispatch", "combine"):
            s["layout"] = nuna.A2ALayout(s["topk"].cpu().numpy(), E).upload()
        if op != "combine":  # kept over many routings: room for every token
            s["recv"] = buffers(P * T, H)
        if op in ("combine", "step"):
            s["out"] = buffers(T, H)
        if op == "routed":
            s["rows"] = torch.zeros(P + 1, dtype=torch.int64, device="cuda")
    return s


def run(s):
    case = s["case"]
    op = case["op"]
    if op == "allreduce":
        if case["prepared"]:
            s["call"]()
            return s["out"]
        return nuna.allreduce(s["in"], s["out"])
    if op == "reduce_scatter":
        return nuna.reduce_scatter(s["in"], s["out"])
    if op == "all_gather":
        return nuna.all_gather(s["in"], s["out"])
    if op == "dispatch":
        return nuna.all_to_all(s["send"], s["recv"], s["layout"])
    if op == "combine":
        return nuna.all_to_all_combine(s["y"], s["out"], s["layout"], weights=s["weights"])
    if op == "routed":
        return nuna.all_to_all_routed(s["send"], s["recv"], s["topk"], case["experts"], s["rows"]), s["rows"]
    # One step: the gate kernel's table comes to the host, the layout is planned and uploaded, and the rows go
    # out and come back (the experts between are not part of this framework; they return the rows unchanged).
    # A layout may be freed only when no enqueued call uses it.
    layout = nuna.A2ALayout(s["topk"].cpu().numpy(), case["experts"]).upload()
    nuna.all_to_all(s["send"], s["recv"], layout)
    nuna.all_to_all_combine(s["recv"], s["out"], layout)
    torch.cuda.current_stream().synchronize()
    layout.close()
    return s["recv"], s["out"]


def _expected_rows(case):
    """Rows received over all ranks: each token goes once to every distinct rank of its k of E experts."""
    E, k, P = case["experts"], case["topk"], case["ranks"]
    return P * case["tokens"] * P * (1.0 - math.comb(E - E // P, k) / math.comb(E, k))


def work(case):
    op, P, es = case["op"], case["ranks"], ESIZE[case["dtype"]]
    if op == "allreduce":
        return {"bytes": 2 * P * case["count"] * es, "flops": (P - 1) * case["count"]}
    if op == "reduce_scatter":
        return {"bytes": (P + 1) * P * case["count"] * es, "flops": (P - 1) * P * case["count"]}
    if op == "all_gather":
        return {"bytes": (P + 1) * P * case["count"] * es, "flops": 0}
    H, rows, tokens = case["hidden"], _expected_rows(case), P * case["tokens"]
    once = (rows + tokens) * H * es
    if op == "dispatch":
        return {"bytes": once, "flops": 0}
    if op == "routed":
        return {"bytes": once + 4 * tokens * case["topk"], "flops": 0}
    if op == "combine":
        return {"bytes": once + (4 * rows if case["weighted"] else 0),
                "flops": (2 if case["weighted"] else 1) * rows * H}
    return {"bytes": 2 * once + 4 * tokens * case["topk"], "flops": rows * H}


def tolerance(case):
    return "exact"


def _sent(case, topk):
    """bool [P * T, P]: token (source-major) goes to rank."""
    P = case["ranks"]
    ranks = (topk.long() // (case["experts"] // P)).reshape(P * case["tokens"], -1)
    return torch.zeros((P * case["tokens"], P), dtype=torch.bool, device=topk.device).scatter_(1, ranks, True)


def exact(case, seed):
    s = _inputs(case, seed)
    op, P = case["op"], case["ranks"]
    if op in ("allreduce", "reduce_scatter"):
        total = s["in"][0].double()
        for t in s["in"][1:]:
            total += t.double()
        if op == "allreduce":
            return [total] * P
        return list(total.view(P, -1))
    if op == "all_gather":
        return [torch.cat(s["in"]).double()] * P
    T, H = case["tokens"], case["hidden"]
    sent = _sent(case, s["topk"])
    at = sent.long().cumsum(dim=0) - 1  # receive row of token i at rank d
    if op == "combine":
        out = torch.zeros((P * T, H), dtype=torch.float64, device="cuda")
        for d in range(P):
            tok = sent[:, d].nonzero().squeeze(1)
            term = s["y"][d][at[tok, d]].double()
            if case["weighted"]:
                term *= s["weights"].view(P * T, P)[tok, d].double().unsqueeze(1)
            out[tok] += term
        return list(out.view(P, T, H))
    send = torch.cat(s["send"])
    recv = []
    for d in range(P):
        r = torch.zeros((P * T, H), dtype=torch.float64, device="cuda")
        tok = sent[:, d].nonzero().squeeze(1)
        r[at[tok, d]] = send[tok].double()
        recv.append(r)
    if op == "dispatch":
        return recv
    if op == "routed":
        return recv, None
    back = send.double() * sent.sum(dim=1, keepdim=True)
    return recv, list(back.view(P, T, H))
