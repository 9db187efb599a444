"""The calls a user of this library makes, as measurable cases.

A rank of an expert-parallel model counts its routing (``demand``), plans the AlltoAllv (``plan``,
``Pipeline.step``), packs its rows or heads into the send buffer, and takes the returned rows back
(``unpack_rows``, ``pack_combine``, ``unpack_combine``); a serving loop plans several matrices ahead
(``plan_batch``).  The listed sizes are the library's named workloads, from an eight-GPU node to 256
ranks; ``draw`` spreads the same calls over the ranges those workloads span.

All outputs are whole numbers or bytes and do not depend on an order of summation, so every case is exact.
"""
import math
import types

import torch

import paper_2609_34340_amd as vp

PCIE, NIC = 32, 25   # bytes per ns


def listed():
    return [
        # one rank's own routing in a decode step, 64-rank expert parallelism: the smallest call, all launch latency
        dict(name="demand-decode", kind="demand", nodes=8, ranks="one", tokens=96, hidden=4096, experts=256, top_k=8,
             law="zipf", skew=1.0),
        # every rank's routing of a prefill layer at 64 ranks (the planner's input on one GPU)
        dict(name="demand-prefill-64", kind="demand", nodes=8, ranks="all", tokens=16384, hidden=4096, experts=256,
             top_k=8, law="zipf", skew=1.0),
        # demand -> control words -> plan -> pack, one eight-GPU node, uniform top-2 routing
        dict(name="step-moe-8", kind="step", nodes=1, tokens=2048, hidden=2048, experts=32, top_k=2, law="uniform",
             skew=0.0),
        # the same step on two nodes: prefill of a 128-expert top-8 model with skewed experts
        dict(name="step-moe-16", kind="step", nodes=2, tokens=8192, hidden=2048, experts=128, top_k=8, law="zipf",
             skew=1.2),
        # the same step at 256 ranks, 14 KiB rows, a hot tenth of the experts: the largest
        dict(name="step-moe-256", kind="step", nodes=32, tokens=4096, hidden=7168, experts=256, top_k=8, law="hot",
             skew=0.5),
        # sequence parallelism: 40 heads of 128 unevenly over 16 ranks
        dict(name="step-heads-16", kind="step_heads", nodes=2, tokens=2048, heads=40, head_dim=128),
        # planning alone: the 64-rank prefill matrix
        dict(name="plan-moe-64", kind="plan", nodes=8, demand="moe", tokens=16384, unit=8192, experts=256, top_k=8,
             law="zipf", skew=1.0),
        # planning alone: a skewed AlltoAllv of 1 GiB per source on nodes with cross-socket peer to peer
        dict(name="plan-skew-sys-16", kind="plan", nodes=2, sys=True, demand="pairs", per_rank=1 << 30, unit=4096,
             skew=0.6),
        # a stream of sixteen 64-rank matrices planned ahead, side by side
        dict(name="plan-batch-64", kind="plan_batch", nodes=8, batch=16, demand="moe", tokens=16384, unit=8192,
             experts=256, top_k=8, law="zipf", skew=1.0),
        # packing alone: 8 KiB rows, 1 GiB of send buffer
        dict(name="pack-rows-64", kind="pack_rows", nodes=8, tokens=16384, hidden=4096, experts=256, top_k=8,
             law="zipf", skew=1.0),
        # packing alone: one node's head re-layout of a 75,600-token video sequence (9,450 tokens per rank)
        dict(name="pack-heads-8", kind="pack_heads", nodes=1, tokens=9450, heads=40, head_dim=128),
        # the receive side and the way back of one layer: unpack the dispatch, pack the combine, unpack the combine
        dict(name="return-16", kind="return", nodes=2, tokens=8192, hidden=2048, experts=128, top_k=8, law="zipf",
             skew=1.2),
    ]


# ------------------------------------------------------------------ drawn cases

def _log(rng, lo, hi):
    return int(min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def _law(rng):
    law = rng.choice(["uniform", "zipf", "zipf", "hot"])
    return dict(law=law, skew={"uniform": 0.0, "zipf": round(rng.uniform(0.3, 1.4), 2), "hot": 0.5}[law])


def _moe(rng, max_nodes, max_ids, max_send):
    """A MoE layer: nodes, tokens, top-k, experts and row size; `max_ids` bounds all ranks' assignments, `max_send`
    one rank's send buffer."""
    nodes = _log(rng, 1, max_nodes)
    n = 8 * nodes
    top_k = rng.choice([1, 2, 4, 6, 8])
    experts = n * rng.choice([e for e in (1, 2, 3, 4, 8, 16) if 2 * top_k <= n * e <= 512])
    hidden = 8 * _log(rng, 32, 1024)
    most = min(16384, max_ids // (n * top_k), max_send // (top_k * hidden * 2))
    return dict(nodes=nodes, k_per_rank=16, tokens=_log(rng, 1, max(1, most)), hidden=hidden, experts=experts, top_k=top_k, **_law(rng))


def draw(rng):
    kind = rng.choice(["demand", "step", "step", "step_heads", "plan", "plan", "plan_batch", "pack_rows", "pack_heads",
                       "return"])
    ids = 8 << 20
    if kind == "demand":
        return dict(kind=kind, ranks=rng.choice(["one", "all"]), **_moe(rng, 32, ids, 1 << 40))
    if kind == "step":
        return dict(kind=kind, **_moe(rng, 32, ids, 400 << 20))
    if kind == "pack_rows":
        return dict(kind=kind, **_moe(rng, 8, ids, 1 << 30))
    if kind == "return":
        return dict(kind=kind, **_moe(rng, 4, ids, 128 << 20))
    if kind in ("step_heads", "pack_heads"):
        nodes = _log(rng, 1, 4)
        return dict(kind=kind, nodes=nodes, k_per_rank=16, tokens=_log(rng, 1, 9450), heads=_log(rng, 4 * nodes, 64),
                    head_dim=8 * _log(rng, 4, 32))
    if kind == "plan_batch":
        case = dict(kind=kind, k_per_rank=16, nodes=_log(rng, 1, 8), batch=_log(rng, 2, 32))
    else:
        case = dict(kind=kind, k_per_rank=16)
        shape = rng.choice(["standard", "standard", "sys", "four", "three", "nics"])
        if shape == "standard":
            case.update(nodes=_log(rng, 1, 32))
        elif shape == "sys":
            case.update(nodes=_log(rng, 1, 16), sys=True)
        elif shape == "four":     # two switches of four GPUs, on one socket or two
            case.update(nodes=_log(rng, 1, 16), gpus=4, **rng.choice([dict(sockets=1), dict(switches=1)]))
        elif shape == "three":
            case.update(nodes=_log(rng, 1, 16), gpus=3, sockets=1)
        else:
            case.update(nodes=_log(rng, 1, 4), nics=2, sockets=1)
    n = _topo(case)[1]
    if rng.random() < 0.6:
        case.update(demand="moe", experts=n * rng.choice([1, 2, 4]) if n < 128 else n, top_k=rng.choice([2, 4, 8]),
                    tokens=_log(rng, 256, max(256, min(8192, ids // (8 * n)))), unit=16 * _log(rng, 16, 1024), **_law(rng))
        case["top_k"] = min(case["top_k"], case["experts"] // 2)
    else:
        case.update(demand="pairs", per_rank=_log(rng, 16 << 20, 1 << 30), unit=4096, skew=round(rng.uniform(0.0, 0.9), 2))
    return case


# ------------------------------------------------------------------ inputs

def _topo(case):
    t = types.SimpleNamespace(n_nodes=case["nodes"], sockets_per_node=case.get("sockets", 2),
                              switches_per_socket=case.get("switches", 2), gpus_per_switch=case.get("gpus", 2),
                              nics_per_switch=case.get("nics", 1), flags=1 if case.get("sys") else 0,
                              pcie_bytes_per_ns=PCIE, nic_bytes_per_ns=NIC)
    return t, t.n_nodes * t.sockets_per_node * t.switches_per_socket * t.gpus_per_switch


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _popularity(case, gen):
    """Log-probability of every expert: uniform, Zipf over a random order, or half the mass on a hot tenth."""
    e = case["experts"]
    order = torch.randperm(e, generator=gen, device="cuda")
    p = torch.empty(e, device="cuda")
    if case["law"] == "zipf":
        p[order] = torch.arange(1, e + 1, device="cuda", dtype=torch.float32) ** -case["skew"]
    elif case["law"] == "hot":
        hot = max(1, round(0.1 * e))
        p.fill_((1.0 - case["skew"]) / max(1, e - hot))
        p[order[:hot]] = case["skew"] / hot
    else:
        p.fill_(1.0 / e)
    return p.log()


def _routing(case, rows, gen, logp):
    """int32 [rows, T, k]: distinct experts of each token, weighted by popularity (Gumbel top-k)."""
    t, k, e = case["tokens"], case["top_k"], case["experts"]
    out = torch.empty((rows * t, k), dtype=torch.int32, device="cuda")
    for lo in range(0, rows * t, 1 << 17):
        hi = min(rows * t, lo + (1 << 17))
        u = torch.empty((hi - lo, e), device="cuda").exponential_(generator=gen)
        out[lo:hi] = torch.topk(logp - u.log(), k, dim=1).indices
    return out.view(rows, t, k)


def _bf16(shape, gen):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.bfloat16)


def _matrix(case, n, gen):
    """int64 [N, N] byte demand without the library: counted routing, or pairwise Zipf volumes."""
    unit = case["unit"]
    if case["demand"] == "moe":
        r = _routing(case, n, gen, _popularity(case, gen)).view(n, -1).long() // (case["experts"] // n)
        units = torch.zeros((n, n), dtype=torch.int64, device="cuda")
        units.scatter_add_(1, r, torch.ones_like(r))
    else:
        w = torch.arange(1, n, device="cuda", dtype=torch.float64) ** -case["skew"]
        vol = torch.floor(w / w.sum() * (case["per_rank"] // unit)).long()
        units = torch.zeros((n, n), dtype=torch.int64, device="cuda")
        for i in range(n):
            d = torch.randperm(n - 1, generator=gen, device="cuda")
            units[i, d + (d >= i)] = vol
    units.fill_diagonal_(0)
    return units * unit


def _head_split(heads, n):
    """First head of each rank: as even as possible, the larger shares last."""
    base, extra = divmod(heads, n)
    share = torch.full((n,), base, dtype=torch.int64)
    if extra:
        share[n - extra:] += 1
    return torch.cat([torch.zeros(1, dtype=torch.int64), share.cumsum(0)]).cuda()


def _k_max(case, n):
    """Schedule capacity: the library's default of 8 N, more where a drawn demand may need it."""
    return case.get("k_per_rank", 8) * n


def _zeroed(d):
    for v in d.values():
        v.zero_()
    return d


def _schedule(case, n):
    return _zeroed(vp.alloc_schedule(n, _k_max(case, n), layout=True))


def _demand_out(case, rows, n):
    ids = case["tokens"] * case["top_k"]
    return dict(counts=torch.zeros((rows, case["experts"]), dtype=torch.int32, device="cuda"),
                demand=torch.zeros((rows, n), dtype=torch.int64, device="cuda"),
                sorted_tok=torch.zeros(ids, dtype=torch.int32, device="cuda"),
                sorted_slot=torch.zeros(ids, dtype=torch.uint8, device="cuda"),
                dest_off=torch.zeros(n + 1, dtype=torch.int64, device="cuda"))


def _demand_ws(case, rows):
    return torch.zeros(max(1, vp.demand_workspace_bytes(rows, case["tokens"], case["top_k"], case["experts"])),
                       dtype=torch.uint8, device="cuda")


def _planned(case, cat, d, unit):
    """The schedule (with layout) a program has in hand before it packs."""
    p = vp.plan_params(cat.N, unit, k_max=_k_max(case, cat.N))
    s = vp.plan(cat, d, p, out=_schedule(case, cat.N))
    s.pop("status")
    return s


def _bytes_for(send_rows, row):
    return torch.zeros(max(1, send_rows) * row, dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    topo, n = _topo(case)
    gen, kind = _gen(seed), case["kind"]
    s = types.SimpleNamespace(kind=kind, n=n, case=case, status=vp.new_status())
    if kind == "step":
        pipe = vp.Pipeline(topo, "moe", case["hidden"] * 2, n_experts=case["experts"], tokens=case["tokens"],
                           top_k=case["top_k"], params=dict(k_max=_k_max(case, n)))
        s.pipe, s.routing = pipe, _routing(case, n, gen, _popularity(case, gen))
        s.tokens = _bf16((case["tokens"], case["hidden"]), gen)
        _zeroed(pipe.sched), _zeroed(pipe.dem)
        pipe.send.zero_(), pipe.step_off.zero_(), pipe.words.zero_()
        return s
    if kind == "step_heads":
        unit = case["head_dim"] * 2
        pipe = vp.Pipeline(topo, "heads", unit, tokens=case["tokens"], token_stride=case["heads"] * unit,
                           params=dict(k_max=_k_max(case, n)))
        s.pipe, s.head_lo = pipe, _head_split(case["heads"], n)
        s.tokens = _bf16((case["tokens"], case["heads"], case["head_dim"]), gen)
        _zeroed(pipe.sched), _zeroed(pipe.dem)
        pipe.send.zero_(), pipe.step_off.zero_()
        return s
    if kind == "demand":
        s.rows = n if case["ranks"] == "all" else 1
        s.routing = _routing(case, s.rows, gen, _popularity(case, gen))
        s.out, s.ws = _demand_out(case, s.rows, n), _demand_ws(case, s.rows)
        s.words = torch.zeros((s.rows, n), dtype=torch.int32, device="cuda")
        return s
    cat = s.cat = vp.Catalog(topo)
    cat.upload()
    if kind == "plan":
        s.d = _matrix(case, n, gen)
        s.p = vp.plan_params(n, case["unit"], k_max=_k_max(case, n))
        s.out = _schedule(case, n)
        s.ws = torch.zeros(vp.plan_workspace_bytes(cat, s.p), dtype=torch.uint8, device="cuda")
        return s
    if kind == "plan_batch":
        b = case["batch"]
        s.d = torch.stack([_matrix(case, n, gen) for _ in range(b)])
        s.p = vp.plan_params(n, case["unit"], k_max=_k_max(case, n))
        s.out = _zeroed(vp.alloc_schedule_batch(b, n, s.p.k_max, layout=True))
        s.status = torch.zeros(b, dtype=torch.int32, device="cuda")
        s.ws = torch.zeros(vp.plan_batch_workspace_bytes(cat, s.p, b), dtype=torch.uint8, device="cuda")
        return s
    if kind == "pack_heads":
        unit, t = case["head_dim"] * 2, case["tokens"]
        s.head_lo, s.unit, s.stride = _head_split(case["heads"], n), unit, case["heads"] * unit
        s.act = _bf16((t, case["heads"], case["head_dim"]), gen)
        s.sched = _planned(case, cat, vp.demand_heads(t, s.head_lo, unit, R=n), unit)
        s.send = _bytes_for(t * case["heads"], unit)
        s.step_off = torch.zeros(_k_max(case, n) + 1, dtype=torch.int64, device="cuda")
        s.ws = torch.zeros(vp.pack_workspace_bytes(_k_max(case, n), s.send.numel(), unit), dtype=torch.uint8, device="cuda")
        return s
    # pack_rows, return: a routed layer with its demand and schedule in hand
    row, t, k = case["hidden"] * 2, case["tokens"], case["top_k"]
    s.row, s.t, s.k = row, t, k
    s.routing = _routing(case, n, gen, _popularity(case, gen))
    s.dem = vp.demand(s.routing, n, case["experts"], row, out=_demand_out(case, n, n), ws=_demand_ws(case, n))
    s.sched = _planned(case, cat, s.dem["demand"], row)
    s.step_off = torch.zeros(_k_max(case, n) + 1, dtype=torch.int64, device="cuda")
    if kind == "pack_rows":
        s.tokens = _bf16((t, case["hidden"]), gen)
        s.send = _bytes_for(t * k, row)
        s.ws = torch.zeros(vp.pack_workspace_bytes(_k_max(case, n), s.send.numel(), row, t, k), dtype=torch.uint8,
                           device="cuda")
        return s
    # return: receive slots, expert-major output, combine send rows and returned rows of the busiest rank whose
    # rows fit buffers of a fixed capacity (twice the mean)
    cap, slot = 2 * t * k, vp.slot_bytes(row)
    mine = s.dem["counts"].view(n, n, -1).sum((0, 2))
    s.rank = int(torch.where(mine <= cap, mine, -1).argmax())
    s.dem = vp.demand(s.routing, n, case["experts"], row, sort_row=s.rank, out=s.dem, ws=_demand_ws(case, n))
    s.back = _planned(case, cat, vp.demand_transpose(s.dem["demand"]), row)
    s.recv = _bf16((cap * slot // 2,), gen)
    s.expert_out = _bf16((cap * slot // 2,), gen)
    s.out = _bytes_for(cap, slot)
    s.send = _bytes_for(cap, row)
    s.returned = _bf16((t * k * slot // 2,), gen)
    s.combined = torch.zeros((t * k, slot), dtype=torch.uint8, device="cuda")
    s.ws = torch.zeros(vp.unpack_workspace_bytes(cap), dtype=torch.uint8, device="cuda")
    return s


# ------------------------------------------------------------------ one pass

def run(s):
    kind, case = s.kind, s.case
    if kind == "step":
        p = s.pipe
        send = p.step(routing=s.routing, tokens=s.tokens)
        return dict(send=send, step_off=p.step_off, words=p.words, status=p.status, demand=p.dem, sched=p.sched)
    if kind == "step_heads":
        p = s.pipe
        send = p.step(tokens=s.tokens, head_lo=s.head_lo)
        return dict(send=send, step_off=p.step_off, status=p.status, demand=p.dem, sched=p.sched)
    if kind == "demand":
        out = vp.demand(s.routing, s.n, case["experts"], case["hidden"] * 2, status=s.status, out=s.out, ws=s.ws)
        words = vp.control_words(out["counts"], s.n, status=s.status, out=s.words)
        return dict(out, words=words)
    if kind == "plan":
        return vp.plan(s.cat, s.d, s.p, status=s.status, out=s.out, ws=s.ws)
    if kind == "plan_batch":
        return vp.plan_batch(s.cat, s.d, s.p, status=s.status, out=s.out, ws=s.ws)
    if kind == "pack_heads":
        vp.pack_heads(s.act, s.stride, s.head_lo, s.unit, 0, s.sched, s.send, s.step_off, s.status, ws=s.ws)
        return dict(send=s.send, step_off=s.step_off, status=s.status)
    if kind == "pack_rows":
        vp.pack_rows(s.tokens, s.row, s.dem["sorted_tok"], s.dem["sorted_slot"], s.dem["dest_off"], 0, s.sched, s.send,
                     s.step_off, s.status, ws=s.ws)
        return dict(send=s.send, step_off=s.step_off, status=s.status)
    # the dispatch's rows to this rank's experts; the experts' rows back; the returned rows to their tokens
    vp.unpack_rows(s.recv, s.row, s.dem["counts"], s.rank, s.sched, s.out, s.status, ws=s.ws)
    vp.pack_combine(s.expert_out, s.row, s.dem["counts"], s.rank, s.back, s.send, s.step_off, s.status, ws=s.ws)
    vp.unpack_combine(s.returned, s.row, s.t, s.k, s.dem["sorted_tok"], s.dem["sorted_slot"], s.dem["dest_off"], s.rank,
                      s.back, s.combined, s.status, ws=s.ws)
    return dict(out=s.out, send=s.send, combined=s.combined, step_off=s.step_off, status=s.status)


# ------------------------------------------------------------------ what a pass cannot do without

def work(case):
    """Bytes: inputs read once, outputs written once.  A schedule is taken at its target of 2 N activations, each
    lane with destination, instance, bytes, send and stream offsets and receive view (36 bytes).  Operations: one
    counted or compared number each; the path has no floating point."""
    n, kind = _topo(case)[1], case["kind"]
    b = f = 0
    if kind in ("plan", "plan_batch", "step", "step_heads"):
        one = 8 * n * n + 36 * n * 2 * n
        b += one * case.get("batch", 1)
        f += 2 * n * n * case.get("batch", 1)
    if kind in ("step", "demand"):
        rows = 1 if case.get("ranks") == "one" else n
        ids = case["tokens"] * case["top_k"]
        b += 4 * rows * ids + 4 * rows * case["experts"] + 8 * rows * n + 4 * rows * n + 5 * ids + 8 * (n + 1)
        f += rows * ids
    if kind in ("step", "pack_rows"):
        row, t, k = case["hidden"] * 2, case["tokens"], case["top_k"]
        b += t * row + t * k * row * (n - 1) // n + 5 * t * k
    if kind in ("step_heads", "pack_heads"):
        b += 2 * case["tokens"] * case["heads"] * case["head_dim"] * 2 * (n - 1) // n
    if kind == "return":
        rows = case["tokens"] * case["top_k"] * (n - 1) // n
        b += 3 * 2 * rows * case["hidden"] * 2
    return dict(bytes=b, flops=f)


def tolerance(case):
    return "exact"


def exact(case, seed):
    """The demand outputs in plain torch; the other cases' outputs follow from the planner's choices or are copies."""
    if case["kind"] != "demand":
        return None
    n = _topo(case)[1]
    gen = _gen(seed)
    rows = n if case["ranks"] == "all" else 1
    routing = _routing(case, rows, gen, _popularity(case, gen)).view(rows, -1).long()
    e, k, unit = case["experts"], case["top_k"], case["hidden"] * 2
    per = e // n
    counts = torch.zeros((rows, e), dtype=torch.int64, device="cuda").scatter_add_(1, routing, torch.ones_like(routing))
    d = counts.view(rows, n, per).sum(2) * unit
    d[torch.arange(rows), torch.arange(rows)] = 0
    order = torch.sort(routing[0], stable=True).indices
    off = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), counts[0].view(n, per).sum(1).cumsum(0)])
    return dict(counts=counts.int(), demand=d, sorted_tok=(order // k).int(), sorted_slot=(order % k).to(torch.uint8),
                dest_off=off, words=None, status=torch.zeros(1, dtype=torch.int32))
