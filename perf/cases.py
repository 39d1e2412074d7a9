"""The work that programs built on this package have it do, as measurable cases.

A program that looks for a good device partition of a data-flow graph packs the graph once
(CpGraph), keeps its output tensors and workspaces, and then calls, over and over with new
candidate partitions: cp_eval (critical path, levels and mask of a batch), cp_pct_order (priority
lists), cp_critical_path (one path per partition), cp_simulate (list scheduling), cp_search (descent
from a start) and cp_seed_partition (the start).  The graphs are the synthetic families of this
repository's workloads: layered random graphs, a sharded multilayer perceptron with its backward
mirror, inception-like modules with their mirror, and wide levels with hubs.

All outputs are whole numbers, so every tolerance is "exact".
"""
from __future__ import annotations

import ctypes

import numpy as np
import torch

import paper_1711_01912_amd as cpe
from paper_1711_01912_amd import binding

DEVICE = "cuda:0"


def listed():
    return [
        # one call of a tight loop: eight levels of eight vertices, where only launches and host time count
        dict(name="eval-tiny", op="eval", graph="layered", levels=8, width=8, deg=3, span=2, k=2, P=16, layout="vertex"),
        # a training step of a sharded perceptron: narrow levels, every forward vertex also read by its backward twin
        dict(name="eval-mlp", op="eval", graph="mlp", levels=32, width=7, k=4, P=1024, layout="partition"),
        # modules of parallel chains with skip edges and backward twins at the far end of the graph, a large batch
        dict(name="eval-inception", op="eval", graph="inception", levels=50, width=14, k=8, P=4096, layout="partition"),
        # the benchmark's workload: a million vertices in two thousand levels
        dict(name="eval-large", op="eval", graph="layered", levels=2000, width=500, deg=7, span=10, k=16, P=256,
             layout="partition"),
        # nothing a multiple of anything, results compared across partitions (one row per vertex)
        dict(name="eval-ragged", op="eval", graph="layered", levels=701, width=173, deg=5, span=6, k=11, P=777,
             layout="vertex"),
        # twenty wide levels, one vertex in a hundred feeding a thousand others
        dict(name="eval-hubs", op="eval", graph="hubs", levels=20, width=10000, deg=1000, k=8, P=1024, layout="vertex"),
        # tensor volumes in bytes: path lengths need 64 bits
        dict(name="eval-bytes-int64", op="eval", graph="layered", levels=301, width=97, deg=4, span=4, k=8, P=320,
             layout="partition", big=True),
        # the priority list of every device, for a batch of partitions of a mid-sized graph
        dict(name="order", op="order", graph="layered", levels=1000, width=211, deg=7, span=10, k=16, P=512,
             layout="partition"),
        # one critical path per partition
        dict(name="path", op="path", graph="layered", levels=701, width=173, deg=5, span=6, k=11, P=777,
             layout="partition"),
        # schedules of a graph of the size the paper simulates, on its fifty devices
        dict(name="simulate-paper", op="simulate", graph="layered", levels=251, width=21, deg=3, span=3, k=50, P=4096,
             layout="partition", policy="pct"),
        # three moves of the descent over moves of critical-path vertices
        dict(name="search", op="search", graph="layered", levels=1000, width=211, deg=7, span=10, k=16, P=1024, moves=3),
        # the paper's Critical Path partition of the same graph, the search's start
        dict(name="seed", op="seed", graph="layered", levels=1000, width=211, deg=7, span=10, k=16, P=1),
    ]


def _log_int(rng, lo, hi):
    """Whole number spread evenly over the logarithm of lo..hi, odd ones among them."""
    return int(min(hi, max(lo, round(2.0 ** rng.uniform(np.log2(lo), np.log2(hi))))))


def draw(rng):
    op = rng.choice(("eval", "eval", "eval", "eval", "eval", "order", "path", "simulate", "search", "seed"))
    k = _log_int(rng, 2, 50)
    if op == "simulate":
        # sequential along every device: thousands of vertices, not millions
        levels = _log_int(rng, 40, 400)
        case = dict(op=op, graph="layered", levels=levels, width=_log_int(rng, 3, max(4, 6000 // levels)), deg=3, span=3,
                    k=k, P=_log_int(rng, 64, 4096), layout="partition", policy=rng.choice(("pct", "fifo")))
        return case
    graph = rng.choice(("layered", "layered", "layered", "mlp", "inception", "hubs"))
    if op in ("search", "seed") and graph == "hubs":
        graph = "layered"
    if graph == "layered":
        n = _log_int(rng, 60, 250_000)
        levels = _log_int(rng, max(8, n // 600), max(9, min(2000, n // 8)))
        case = dict(op=op, graph=graph, levels=levels, width=max(3, n // levels), deg=rng.randint(2, 7),
                    span=rng.randint(1, 10))
        if rng.random() < 0.25:
            case["renumber"] = True       # vertex numbers in no relation to the levels
    elif graph == "mlp":
        case = dict(op=op, graph=graph, levels=_log_int(rng, 4, 64), width=rng.randint(1, 8))
    elif graph == "inception":
        case = dict(op=op, graph=graph, levels=_log_int(rng, 4, 50), width=rng.randint(1, 14))
    else:
        width = _log_int(rng, 1000, 10000)
        case = dict(op=op, graph=graph, levels=rng.randint(8, 20), width=width, deg=width // 10)
    n = _vertices(case)
    most = 16 if graph == "hubs" else 50
    case["k"] = min(k, most)
    if op in ("search", "seed"):
        case["P"] = 1
        if op == "search":
            case["P"], case["moves"] = 1024, rng.randint(1, 3)
        return case
    case["P"] = _log_int(rng, 8, max(16, min(4096, 80_000_000 // n)))
    case["layout"] = rng.choice(("partition", "vertex"))
    if op == "eval" and graph == "layered" and rng.random() < 0.2:
        case["big"] = True
    return case


def _vertices(case):
    a, b = case["levels"], case["width"]
    if case["graph"] == "mlp":
        return 9 * a * b
    if case["graph"] == "inception":
        return 2 * a * (2 + 14 * b)
    return a * b


def _edges(case):
    a, b, n = case["levels"], case["width"], _vertices(case)
    if case["graph"] == "layered":
        return (a - 1) * b * (1 + case["deg"]) // 2
    if case["graph"] == "mlp":
        return 2 * (3 * a * b + (a - 1) * b * b) + 5 * a * b
    if case["graph"] == "inception":
        return 5 * n // 2
    return (a - 1) * (b // 100 * case["deg"] + (b - b // 100) * 3)


# ---- graphs ---------------------------------------------------------------------------------------------------------

def _layered(case, rng):
    """Every vertex but the last level's draws 1..deg out-edges over 1..span levels."""
    levels, width = case["levels"], case["width"]
    n = levels * width
    src = np.repeat(np.arange(n - width), rng.integers(1, case["deg"] + 1, n - width))
    at = src // width
    to = at + 1 + (rng.random(len(src)) * np.minimum(case["span"], levels - 1 - at)).astype(np.int64)
    dst = to * width + rng.integers(0, width, len(src))
    level = np.arange(n) // width
    if case.get("renumber"):
        name = rng.permutation(n)
        src, dst, old = name[src], name[dst], level
        level = np.empty(n, dtype=np.int64)
        level[name] = old
    if case.get("big"):
        t, c = rng.integers(1, 1 << 28, len(src)), rng.integers(1, 1 << 20, n)
    elif case["op"] == "simulate":
        t, c = rng.integers(1, 101, len(src)), rng.integers(1, 101, n)
    else:
        t, c = rng.integers(1, 10001, len(src)), rng.integers(1, 1001, n)
    return n, src, dst, t, c, level


def _mirrored(n, src, dst, t, c_of, t_of):
    """Forward graph, the reversed backward edges, and an edge from every vertex to its backward twin."""
    x = np.arange(n)
    return (2 * n, np.concatenate([src, dst + n, x]), np.concatenate([dst, src + n, x + n]),
            np.concatenate([t, t, t_of(n)]), c_of(2 * n))


def _longest_levels(n, src, dst):
    level = np.zeros(n, dtype=np.int64)
    while True:
        new = level.copy()
        np.maximum.at(new, dst, level[src] + 1)
        if np.array_equal(new, level):
            return level
        level = new


def _mlp(case, rng):
    """Layers of (product, bias, activation, loss branch), each in shards; a product needs every activation before it."""
    layers, g = case["levels"], case["width"]
    ids = np.arange(layers * 4 * g).reshape(layers, 4, g)
    volume = 4 * np.array([256, 512, 1024, 2048, 4096])[np.arange(layers) % 5]
    src = [ids[:, 0], ids[:, 1], ids[:, 2], np.repeat(ids[:-1, 2], g, axis=1)]
    dst = [ids[:, 1], ids[:, 2], ids[:, 3], np.tile(ids[1:, 0], (1, g))]
    t = [np.repeat(volume[:len(s)], s.shape[1]) for s in src]
    src, dst, t = (np.concatenate([x.ravel() for x in v]) for v in (src, dst, t))
    n = ids.size
    per_vertex = np.repeat(volume, 4 * g)
    n, src, dst, t, _ = _mirrored(n, src, dst, t, lambda m: None, lambda m: per_vertex)
    update = n + np.arange(layers * g)      # one weight update per layer and shard, fed by the backward product
    src = np.concatenate([src, (ids[:, 0] + n // 2).ravel()])
    dst = np.concatenate([dst, update])
    t = np.concatenate([t, np.repeat(volume, g)])
    n += len(update)
    return n, src, dst, t, rng.integers(10, 1001, n), _longest_levels(n, src, dst)


def _inception(case, rng):
    """Modules in sequence: split, four branches of `width` chains of 2 to 5 vertices, concat; skip edges inside a module."""
    groups = case["width"]
    src, dst, n, concat = [], [], 0, -1
    for _ in range(case["levels"]):
        split, depth = n, np.repeat(rng.permutation([2, 3, 4, 5]), groups)
        n += 1
        if concat >= 0:
            src.append([concat])
            dst.append([split])
        first = n + np.concatenate([[0], np.cumsum(depth)])
        n = int(first[-1])
        concat, n = n, n + 1
        body = np.arange(split + 1, concat)
        head = np.isin(body, first[:-1])
        src.append(np.where(head, split, body - 1))
        dst.append(body)
        src.append(first[1:] - 1)
        dst.append(np.full(4 * groups, concat))
        place = body - np.repeat(first[:-1], depth)       # position inside its chain
        a, b = rng.integers(0, len(body), (2, 2 * len(body)))
        keep = place[a] < place[b]
        src.append(body[a[keep]])
        dst.append(body[b[keep]])
    src, dst = np.concatenate(src), np.concatenate(dst)
    log_normal = lambda mean, sigma, m: np.maximum(1, np.rint(rng.lognormal(mean, sigma, m))).astype(np.int64)
    n, src, dst, t, c = _mirrored(n, src, dst, log_normal(8.0, 1.5, len(src)), lambda m: log_normal(4.0, 1.0, m),
                                  lambda m: log_normal(8.0, 1.5, m))
    return n, src, dst, t, c, _longest_levels(n, src, dst)


def _hubs(case, rng):
    """Wide levels; one vertex in a hundred feeds `deg` vertices of the next level, the others 2 to 4."""
    levels, width = case["levels"], case["width"]
    n, inner = levels * width, (levels - 1) * width
    out = rng.integers(2, 5, inner)
    out[rng.choice(inner, inner // 100, replace=False)] = case["deg"]
    src = np.repeat(np.arange(inner), out)
    dst = (src // width + 1) * width + rng.integers(0, width, len(src))
    t = np.minimum(1e7, np.floor(100.0 * (1.0 - rng.random(len(src))) ** (-1.0 / 1.2))).astype(np.int64)
    return n, src, dst, t, rng.integers(1, 51, n), np.arange(n) // width


def _host_inputs(case, seed):
    """Graph arrays, cost model and assignments, made from the case and the seed alone."""
    rng = np.random.default_rng([seed, 1711])
    make = {"layered": _layered, "mlp": _mlp, "inception": _inception, "hubs": _hubs}[case["graph"]]
    n, src, dst, t, c, level = make(case, rng)
    by_src = np.argsort(src, kind="stable") if np.any(src[1:] < src[:-1]) else slice(None)
    src, dst, t = src[by_src], dst[by_src], t[by_src]
    by_dst = np.argsort(dst, kind="stable")
    starts = lambda x, m: np.concatenate([[0], np.cumsum(np.bincount(x, minlength=m))]).astype(np.int32)
    k = case["k"]
    paper = case["op"] == "simulate"      # section 5.1's ranges of speeds and rates
    speeds = rng.integers(10, 101, k) if paper else rng.integers(1, 17, k)
    rates = rng.integers(10, 61, (k, k)) if paper else rng.integers(1, 65, (k, k))
    rows = 1 if case["op"] in ("search", "seed") else case["P"]
    host = dict(n=n, succ_ptr=starts(src, n), succ_idx=dst.astype(np.int32), succ_t=t.astype(np.int64),
                pred_ptr=starts(dst, n), pred_idx=src[by_dst].astype(np.int32), pred_eid=by_dst.astype(np.int32),
                c=c.astype(np.int64), level_ptr=starts(level, int(level.max()) + 1),
                level_vtx=np.argsort(level, kind="stable").astype(np.int32))
    return host, speeds.astype(np.int64), rates.astype(np.int64), rng.integers(0, k, (rows, n), dtype=np.uint8)


# ---- cases ----------------------------------------------------------------------------------------------------------

def prepare(case, seed):
    host, speeds, rates, a = _host_inputs(case, seed)
    graph = cpe.CpGraph(**host, device=DEVICE)
    s = dict(op=case["op"], graph=graph, speeds=speeds, rates=rates, k=case["k"], a=torch.from_numpy(a).to(DEVICE))
    n, P, info = host["n"], case["P"], graph.info
    if s["op"] == "search":
        s["start"], s["moves"], s["chunk"] = s["a"][0].contiguous(), case["moves"], P
        return s
    if s["op"] == "seed":
        return s
    layout = cpe.OUT_PARTITION_MAJOR if case["layout"] == "partition" else cpe.OUT_VERTEX_MAJOR
    s["layout"] = layout
    if s["op"] == "eval":
        rows, cols = (n, P) if layout == cpe.OUT_VERTEX_MAJOR else (P, n)
        tick = torch.int32 if info["min_tick_bytes"] == 4 else torch.int64
        new = lambda shape, kind: torch.empty(shape, dtype=kind, device=DEVICE)
        s["out"] = dict(cp=new(P, torch.int64), b=new((rows, cols), tick), tl=new((rows, cols), tick),
                        mask=new((rows, (cols + 63) // 64), torch.int64), status=new(1, torch.int32))
        s["work"] = new(binding.workspace_bytes(graph, P, s["k"], out_layout=layout), torch.uint8)
        return s
    if s["op"] == "simulate" and case["policy"] == "fifo":
        s["policy"], s["b"] = cpe.POLICY_FIFO, None
        s["tie"] = torch.from_numpy(np.random.default_rng([seed, 5]).permutation(n).astype(np.int32)).to(DEVICE)
    else:
        levels = cpe.cp_eval(graph, s["a"], speeds, rates, want=("cp", "b"), out_layout=layout)
        s["policy"], s["b"], s["cp"], s["tie"] = cpe.POLICY_PCT, levels["b"], levels["cp"], None
        s["max_b"] = int(levels["cp"].max())
    if s["op"] == "simulate":
        need = ctypes.c_size_t(0)
        rc = cpe.load_library().cp_simulate_workspace_bytes(graph._handle, P, s["k"], int(s["policy"]),
                                                            int(s["tie"] is not None), ctypes.byref(need))
        assert rc == 0
        s["work"] = torch.empty(need.value, dtype=torch.uint8, device=DEVICE)
    return s


def run(s):
    graph, a = s["graph"], s["a"]
    if s["op"] == "eval":
        cpe.cp_eval(graph, a, s["speeds"], s["rates"], out=s["out"], workspace=s["work"], out_layout=s["layout"],
                    check_status=False)
        return s["out"]
    if s["op"] == "order":
        return cpe.cp_pct_order(graph, a, s["k"], s["b"], max_b=s["max_b"], b_layout=s["layout"], check_status=False)
    if s["op"] == "path":
        return cpe.cp_critical_path(graph, a, s["speeds"], s["rates"], s["b"], s["cp"], b_layout=s["layout"],
                                    check_status=False)
    if s["op"] == "simulate":
        return cpe.cp_simulate(graph, a, s["speeds"], s["rates"], s["policy"], b=s["b"], tie=s["tie"],
                               b_layout=s["layout"], workspace=s["work"], check_status=False)
    if s["op"] == "search":
        return cpe.cp_search(graph, s["start"], s["speeds"], s["rates"], max_moves=s["moves"], chunk=s["chunk"])
    return cpe.cp_seed_partition(graph, s["speeds"])


def work(case):
    """Every input read once, every output written once; an edge costs three whole-number operations per
    partition and sweep (ceil division, sum, maximum).  A step of the search reads the graph for both
    levels of its partition at least once, and so once more for the candidates of the last step."""
    n, m, P, op = _vertices(case), _edges(case), case["P"], case["op"]
    T = 8 if case.get("big") else 4
    structure = 12 * (n + m)
    if op == "eval":
        return {"bytes": structure + n * P * (1 + 2 * T) + n * P // 8 + 8 * P, "flops": 6 * m * P}
    if op == "order":
        return {"bytes": n * P * (1 + T + 4) + 4 * P * (case["k"] + 1), "flops": n * P * max(1, int(np.log2(n)))}
    if op == "path":
        return {"bytes": P * (4 * case["levels"] + 12) + P * case["levels"] * 60, "flops": 16 * P * case["levels"]}
    if op == "simulate":
        return {"bytes": structure + n * P * (1 + 4 + (4 if case["policy"] == "pct" else 0)) + 8 * P,
                "flops": P * (3 * m + 6 * n)}
    if op == "search":
        return {"bytes": (case["moves"] + 1) * (structure + 10 * n), "flops": (case["moves"] + 1) * 6 * m}
    return {"bytes": structure + n, "flops": n * case["k"]}


def tolerance(case):
    return "exact"      # whole numbers


def exact(case, seed):
    """The evaluation level by level in plain 64-bit tensors; the priority lists as one stable sort."""
    if case["op"] not in ("eval", "order") or _vertices(case) * case["P"] > 300_000_000 or case["levels"] > 2000:
        return None
    host, speeds, rates, a = _host_inputs(case, seed)
    on = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(DEVICE)
    ids = on(a.T).contiguous()                                     # [n][P], one row per vertex
    ceil = lambda x, y: -torch.div(-x, y, rounding_mode="floor")
    speed, rate = on(speeds), on(rates)
    n, P = ids.shape
    c, t = on(host["c"]), on(host["succ_t"])
    src = on(np.repeat(np.arange(n), np.diff(host["succ_ptr"])))
    dst = on(host["succ_idx"].astype(np.int64))
    level = np.empty(n, dtype=np.int64)
    L = len(host["level_ptr"]) - 1
    level[host["level_vtx"]] = np.repeat(np.arange(L), np.diff(host["level_ptr"]))

    def sweep(near, far, tail_term):
        """Values from the far end of each edge to the near one, level by level of the near end."""
        value = torch.zeros((n, P), dtype=torch.int64, device=DEVICE)
        where = on(level)
        order = torch.argsort(where[near], stable=True)
        cut = torch.bincount(where[near], minlength=L).cumsum(0).tolist()
        steps = range(L - 1, -1, -1) if not tail_term else range(L)
        for l in steps:
            e = order[(cut[l - 1] if l else 0):cut[l]]
            for part in e.split(max(1, 40_000_000 // P)):
                x, y = near[part], far[part]
                u, v = (y, x) if tail_term else (x, y)
                pu, pv = ids[u].long(), ids[v].long()
                cost = torch.where(pu == pv, 0, ceil(t[part][:, None], rate[pu, pv])) + value[y]
                if tail_term:
                    cost += ceil(c[u][:, None], speed[pu])
                value.scatter_reduce_(0, x[:, None].expand_as(cost), cost, "amax")
            if not tail_term:
                row = on(host["level_vtx"][host["level_ptr"][l]:host["level_ptr"][l + 1]].astype(np.int64))
                value[row] += ceil(c[row][:, None], speed[ids[row].long()])
        return value

    b = sweep(src, dst, False)
    partition = case["layout"] == "partition"
    if case["op"] == "order":
        seg = torch.zeros((P, case["k"] + 1), dtype=torch.int64, device=DEVICE)
        order = torch.empty((P, n), dtype=torch.int64, device=DEVICE)
        for j in range(P):
            p = ids[:, j].long()
            by_b = torch.argsort(b[:, j], descending=True, stable=True)
            order[j] = by_b[torch.argsort(p[by_b], stable=True)]
            seg[j, 1:] = torch.bincount(p, minlength=case["k"]).cumsum(0)
        return order.to(torch.int32), seg.to(torch.int32)
    tl = sweep(dst, src, True)
    cp = b.amax(0)
    bits = tl + b == cp
    shape = lambda x: x.T.contiguous() if partition else x
    bits = shape(bits)
    padded = torch.zeros((bits.shape[0], (bits.shape[1] + 63) // 64 * 64), dtype=torch.int64, device=DEVICE)
    padded[:, :bits.shape[1]] = bits
    mask = (padded.view(bits.shape[0], -1, 64) << torch.arange(64, device=DEVICE)).sum(-1)
    tick = torch.int64 if case.get("big") else torch.int32
    return dict(cp=cp, b=shape(b).to(tick), tl=shape(tl).to(tick), mask=mask,
                status=torch.zeros(1, dtype=torch.int32, device=DEVICE))
