"""The searches that the framework's speed is measured on.

Each case is one whole search as a program asks for it: the forward call and
the plan recovery, through `paper_2504_00598_amd.search` or, for the one-call
forms, `paper_2504_00598_amd._lib`.  Sizes are those of `workloads.configs`
and of the GPU tests, and generic ones between them.

    call        entry point
    "search"    cfp_search_chain (one call, small searches)
    "noalloc"   cfp_search_chain_noalloc (callers that may not allocate)
    "chain"     search.dp_chain
    "mem"       search.dp_chain_mem, one budget per search
    "frontier"  search.mem_frontier, every budget
    "seg"       search.dp_segments
    "scan"      search.minplus_scan

Fields of a case: n blocks (or segments), k strategies (or plans), b searches,
tables (distinct resharding or boundary tables), edges ("layers": edge i uses
table i mod tables, as in a chain of equal layers of `tables` blocks; "kinds":
two kinds of layers, each with half of the tables, every third layer of the
second kind), costs ("own": every block its own; "repeat": one layer's costs
repeated, as when the profile of a matched segment is reused), gaps (share of
strategies that a block does not offer), free (share of strategy pairs without
resharding besides the diagonal), hi (costs and resharding times are uniform in
[10^4, hi)), m (memory buckets) and s (strategies of a segment's
block).
"""
from __future__ import annotations

import math

import torch

from paper_2504_00598_amd import _lib, search

COST_INF = 0x7FFFFFFF
BIG = 1 << 50        # "no plan" inside the 64-bit reference
OPT_NONE = (1 << 63) - 1


def _case(name, call, n, k, b, tables=12, edges="layers", costs="own", gaps=0.0, free=0.0, hi=1_000_000,
          m=0, s=0):
    return {"name": name, "call": call, "n": n, "k": k, "b": b, "tables": tables, "edges": edges, "costs": costs,
            "gaps": gaps, "free": free, "hi": hi, "m": m, "s": s}


def listed():
    return [
        # one small model, one search: latency of a single call
        _case("search_n24_k16", "search", 24, 16, 1),
        # one model of 24 layers of 12 blocks planned inside a serving loop that may not allocate
        _case("noalloc_n288_k64", "noalloc", 288, 64, 1),
        # 96 layers of 12 blocks, 64 strategies, a sweep of 256 cost tables (batch and hardware variants)
        _case("chain_n1152_k64_b256", "chain", 1152, 64, 256, hi=10_000_000),
        # the same depth with few strategies (3^3) and a small sweep; layers repeat one profile
        _case("chain_n1152_k27_b32", "chain", 1152, 27, 32, costs="repeat"),
        # two kinds of layers (dense and expert), 81 strategies of which some blocks offer fewer, ragged length
        _case("chain_n393_k81_b24", "chain", 393, 81, 24, tables=16, edges="kinds", gaps=0.1),
        # wide strategy space with many free transitions, a sweep of 64
        _case("chain_n512_k256_b64", "chain", 512, 256, 64, free=0.25, hi=10_000_000),
        # the deepest chain and the widest strategy space, few searches
        _case("chain_n4096_k512_b4", "chain", 4096, 512, 4),
        # memory-constrained planning: 24 layers, 1024 buckets, 16 budgets
        _case("mem_n288_k32_b16", "mem", 288, 32, 16, m=1024),
        # the cost-against-memory curve of one model at an odd size
        _case("frontier_n97_k45_b3", "frontier", 97, 45, 3, tables=10, gaps=0.1, m=777),
        # segment-level search, a sweep of 256
        _case("seg_n96_k81_b256", "seg", 96, 81, 256, tables=2, hi=10_000_000, s=3),
        # segment-level search of one model with many plans per segment
        _case("seg_n50_k216_b2", "seg", 50, 216, 2, tables=2, costs="repeat", hi=10_000_000, s=6),
        # the scan form on the deepest chain: the largest job
        _case("scan_n4096_k512_b4", "scan", 4096, 512, 4),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    case = _drawn(rng)
    del case["name"]
    return case


def _drawn(rng):
    call = rng.choice(["search", "noalloc", "chain", "chain", "chain", "chain", "mem", "frontier", "seg", "seg",
                       "scan"])
    tables = rng.choice([1, 2, 4, 6, 10, 12, 12, 12, 16, 24])
    edges = "kinds" if tables >= 4 and tables % 2 == 0 and rng.random() < 0.4 else "layers"
    costs = rng.choice(["own", "own", "repeat"])
    gaps, free = rng.choice([0.0, 0.0, 0.1]), rng.choice([0.0, 0.0, 0.25])
    hi = rng.choice([1_000_000, 5_000_000])
    if call == "search":
        return _case("", call, _log(rng, 8, 72), _log(rng, 3, 20), _log(rng, 1, 32), min(tables, 12), edges, costs,
                     gaps, free, hi)
    if call == "noalloc":
        k = _log(rng, 8, 160)
        n = min(_log(rng, 24, 1152), 24000 // k)
        return _case("", call, n, k, rng.choice([1, 1, 2, 4]), tables, edges, costs, gaps, free, hi)
    if call == "chain":
        k, n, b = _log(rng, 6, 512), _log(rng, 24, 4096), _log(rng, 1, 256)
        b = max(1, min(b, 4_400_000_000 // (n * k * k)))
        return _case("", call, n, k, b, tables, edges, costs, gaps, free, hi)
    if call in ("mem", "frontier"):
        k, n, m, b = _log(rng, 6, 128), _log(rng, 24, 400), _log(rng, 64, 1200), _log(rng, 1, 16)
        b = max(1, min(b, 6_000_000_000 // (n * k * k * m)))
        return _case("", call, n, k, b, min(tables, 12), edges, costs, gaps, free, 1_000_000, m)
    if call == "seg":
        s, p = rng.choice([(3, 4), (3, 3), (4, 3), (2, 5), (6, 3), (5, 3), (2, 7), (7, 2), (3, 5), (8, 3), (4, 4)])
        return _case("", call, _log(rng, 12, 384), s ** p, _log(rng, 1, 512), rng.choice([1, 2, 4]), "layers", costs,
                     gaps, 0.0, hi, 0, s)
    k, n, b = _log(rng, 24, 512), _log(rng, 48, 4096), rng.choice([1, 2, 4])
    n = max(32, min(n, 400_000_000_000 // (b * k ** 3)))
    return _case("", call, n, k, b, tables, edges, costs, gaps, free, 1_000_000)


def _edges(case):
    """Host edge map: table of the edge from block i-1 to block i."""
    n, e = case["n"], case["tables"]
    if case["call"] == "seg":  # the boundary after the first segment, then those between repeated segments
        return [0, 0][:n] + [1 + (i % (e - 1)) if e > 1 else 0 for i in range(n - 2)]
    if case["edges"] == "kinds":
        h = e // 2
        return [i % h + (h if (i // h) % 3 == 2 else 0) for i in range(n)]
    return [i % e for i in range(n)]


def _inputs(case, seed):
    """The tables of a case: int32 costs, resharding (or boundary) tables with a
    zero diagonal, and for the memory forms uint8 memory and int32 budgets."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    n, k, b, e, hi = (case[x] for x in ("n", "k", "b", "tables", "hi"))

    def rand(shape, lo, top):
        return torch.randint(lo, top, shape, generator=g, device="cuda", dtype=torch.int32)

    period = min(n, e) if case["costs"] == "repeat" else n
    seg = case["call"] == "seg"
    rows = rand((b, period, k), 40_000 if seg else 10_000, 4 * hi if seg else hi)
    if case["gaps"]:  # strategy 0 is always offered
        hole = torch.rand((b, period, k), generator=g, device="cuda") < case["gaps"]
        hole[:, :, 0] = False
        rows = torch.where(hole, torch.full_like(rows, COST_INF), rows)
    at = torch.arange(n, device="cuda") % period
    out = {"cost": rows[:, at].contiguous(), "redge": _edges(case)}
    side = case["s"] if seg else k
    tab = rand((e, side, side), 10_000, hi)
    if case["free"]:
        tab[torch.rand((e, side, side), generator=g, device="cuda") < case["free"]] = 0
    tab.diagonal(dim1=1, dim2=2).zero_()
    out["tab"] = tab
    if seg:
        t = torch.arange(k, device="cuda")
        out["last"] = (t // (k // side)).to(torch.uint8)
        out["first"] = (t % side).to(torch.uint8)
    if case["m"]:
        mrows = rand((b, period, k), 0, 9).to(torch.uint8)
        out["mem"] = mrows[:, at].contiguous()
        m = case["m"]
        out["budget"] = torch.tensor([m - 1 - (m // 32) * (i % 16) for i in range(b)], dtype=torch.int32,
                                     device="cuda")
    return out


def prepare(case, seed):
    d = _inputs(case, seed)
    d["call"], d["m"] = case["call"], case["m"]
    if case["call"] in ("search", "noalloc"):
        d["desc"] = _lib.Desc(d["cost"], d["tab"], d["redge"])
    return d


def run(state):
    call = state["call"]
    if call == "search":
        return _lib.cfp_search_chain(state["desc"])
    if call == "noalloc":
        return _lib.cfp_search_chain_noalloc(state["desc"])
    if call == "chain":
        r = search.dp_chain(state["cost"], state["tab"], state["redge"])
    elif call == "scan":
        r = search.minplus_scan(state["cost"], state["tab"], state["redge"])
    elif call == "seg":
        r = search.dp_segments(state["cost"], state["tab"], state["last"], state["first"], state["redge"])
    elif call == "mem":
        r = search.dp_chain_mem(state["cost"], state["tab"], state["redge"], state["mem"], state["m"],
                                state["budget"])
    else:
        frontier, status, plan, _ = search.mem_frontier(state["cost"], state["tab"], state["redge"], state["mem"],
                                                        state["m"])
        return frontier, status, plan
    return r.opt, r.status, r.plan


def work(case):
    """Inputs read once, results written once; one add and one minimum per cell
    of the recurrence.  The memory form needs only the buckets within each
    budget, a segment step K + L F cells, and the scan form is the composition
    of N transfer matrices (N-1 products of K^3 cells per search)."""
    n, k, b, e, m = (case[x] for x in ("n", "k", "b", "tables", "m"))
    side = case["s"] if case["call"] == "seg" else k
    size = 4 * b * n * k + 4 * e * side * side + 4 * n + 12 * b + 4 * b * n
    cells = b * (n - 1) * k * k
    if case["call"] == "seg":
        cells = b * (n - 1) * (k + side * side)
    elif case["call"] == "scan":
        cells *= k
    elif case["call"] == "mem":
        size += b * n * k + 4 * b
        cells = (n - 1) * k * k * sum(m - (m // 32) * (i % 16) for i in range(b))
    elif case["call"] == "frontier":
        size += b * n * k + 8 * b * (m - 1)
        cells *= m
    return {"bytes": size, "flops": 2 * cells}


def tolerance(case):
    # integers throughout: one optimum, and one plan by the lowest-index rule
    return "exact"


def _lowest(values, dim):
    """Minimum along dim and the lowest index that attains it (values below 2^52)."""
    size = values.shape[dim]
    shape = [1] * values.dim()
    shape[dim] = size
    index = torch.arange(size, device=values.device).reshape(shape)
    packed = (values * size + index).min(dim=dim).values
    return packed // size, packed % size


def exact(case, seed):
    """The recurrence row by row in 64-bit integers."""
    if case["call"] != "scan" and case["b"] * case["n"] * case["k"] ** 2 * max(case["m"], 1) > 2e11:
        return None
    d = _inputs(case, seed)
    n, k, b, m = case["n"], case["k"], case["b"], case["m"]
    dev = d["cost"].device
    tab = d["tab"].to(torch.int64)
    if case["call"] == "seg":
        tab = tab[:, d["last"].long()][:, :, d["first"].long()]

    def row(i):
        c = d["cost"][:, i].to(torch.int64)
        return torch.where(c == COST_INF, torch.full_like(c, BIG), c)

    if not m:
        val = row(0)
        args = torch.zeros((n, b, k), dtype=torch.int16, device=dev)
        for i in range(1, n):
            best, arg = _lowest(val[:, :, None] + tab[d["redge"][i]][None], 1)
            args[i] = arg.to(torch.int16)
            val = torch.clamp(best + row(i), max=BIG)
        opt, state = _lowest(val, 1)
        ok = opt < BIG
        plan = torch.empty((b, n), dtype=torch.int64, device=dev)
        for i in range(n - 1, -1, -1):
            plan[:, i] = state
            state = args[i].gather(1, state[:, None])[:, 0].to(torch.int64)
    else:
        bucket = torch.arange(m, device=dev)
        mem = d["mem"].to(torch.int64)
        budget = (torch.full((b,), m - 1, device=dev, dtype=torch.int64) if case["call"] == "frontier"
                  else d["budget"].to(torch.int64))

        def shifted(p, i, fill):  # p[b][s][m - mem[b][i][s]], fill below bucket 0
            at = bucket[None, None, :] - mem[:, i, :, None]
            return torch.where(at >= 0, p.gather(2, at.clamp(min=0)), torch.full_like(p, fill))

        val = torch.clamp(shifted(torch.zeros((b, k, m), dtype=torch.int64, device=dev), 0, BIG) + row(0)[:, :, None],
                          max=BIG)
        args = torch.zeros((n, b, k, m), dtype=torch.int16, device=dev)
        for i in range(1, n):
            best, arg = _lowest(val[:, :, None, :] + tab[d["redge"][i]][None, :, :, None], 1)
            args[i] = shifted(arg, i, 0).to(torch.int16)
            val = torch.clamp(shifted(best, i, BIG) + row(i)[:, :, None], max=BIG)
        low, final = _lowest(val, 1)
        opt = low.gather(1, budget[:, None])[:, 0]
        ok = opt < BIG
        state, left = final.gather(1, budget[:, None])[:, 0], budget
        plan = torch.empty((b, n), dtype=torch.int64, device=dev)
        each = torch.arange(b, device=dev)
        for i in range(n - 1, -1, -1):
            plan[:, i] = state
            prev = args[i][each, state, left].to(torch.int64)
            left = (left - mem[each, i, state]).clamp(min=0)
            state = prev
        if case["call"] == "frontier":
            opt = torch.where(low < BIG, low, torch.full_like(low, OPT_NONE))
    if case["call"] != "frontier":
        opt = torch.where(ok, opt, torch.full_like(opt, OPT_NONE))
    status = torch.where(ok, 0, 1).to(torch.int32)
    plan = torch.where(ok[:, None], plan, torch.full_like(plan, -1)).to(torch.int32)
    return opt, status, plan
