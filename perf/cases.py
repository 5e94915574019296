"""The work that a program using this library has it do, as measurable cases.

A case is a dict of plain values.  Its "task" says which public entry points a
pass goes through:

  stage2      R.stage2: sample, classify, evaluate, gradient, estimate
  autograd    R.rsr_probability forward and backward (binary components)
  montecarlo  plain Monte Carlo without reference states: R.rsr_sample,
              R.rsr_eval_unknown of every sample, R.rsr_importance
  count       R.rsr_classify in COUNT mode with match counts
  plan        R.Plan.run and results over hazard scenarios of several networks
  stage1      R.stage1 from empty reference sets

`kind` is the system function ("st", "global", "flow"), `nodes` / `edges` the
network, `K` the states per component, `level` the target level (the demand
for max flow), `rows` the reference rows per side, `N` the samples.  Networks
and row pools depend on the sizes alone, as the reference states of a network
do; the component probabilities (the hazard scenario), the choice of rows
from the pool and the sample key come from the seed.
"""
import functools
import math

import numpy as np
import torch

import paper_2604_17066_amd as R


def listed():
    return [
        # The smallest call: a 12-node network, as in an interactive session
        # or a unit test; launches and host latency are what it costs.
        {"name": "step_small", "task": "stage2", "kind": "st", "nodes": 12, "edges": 20, "K": 2,
         "level": 1, "rows": 60, "N": 10_000},
        # The flagship step: single-OD connectivity of a 119-node / 295-edge
        # network, 1e4 rows per side, 1e6 samples.
        {"name": "step_graph2", "task": "stage2", "kind": "st", "nodes": 119, "edges": 295, "K": 2,
         "level": 1, "rows": 10_000, "N": 1_000_000},
        # Three-state components, the bottleneck level 1 (590 bits a sample).
        {"name": "step_multistate", "task": "stage2", "kind": "st", "nodes": 119, "edges": 295,
         "K": 3, "level": 1, "rows": 25_000, "N": 1_000_000},
        # Ragged sizes: an odd sample count that no wide load divides.
        {"name": "step_ragged", "task": "stage2", "kind": "st", "nodes": 186, "edges": 465, "K": 2,
         "level": 1, "rows": 4_999, "N": 250_007},
        # The largest network of the batched study with many rows.
        {"name": "step_wide", "task": "stage2", "kind": "st", "nodes": 500, "edges": 1250, "K": 2,
         "level": 1, "rows": 40_000, "N": 262_144},
        # Global connectivity with reference rows grown by Stage 1: many
        # samples stay unclassified and are evaluated.
        {"name": "step_global", "task": "stage2", "kind": "global", "nodes": 59, "edges": 262,
         "K": 2, "level": 2, "rows": 4_000, "N": 262_144},
        # Maximum flow >= 2 with three-state capacities, rows from Stage 1.
        {"name": "step_flow", "task": "stage2", "kind": "flow", "nodes": 119, "edges": 295, "K": 3,
         "level": 2, "rows": 5_000, "N": 500_000},
        # Differentiable probability inside an optimisation loop.
        {"name": "autograd", "task": "autograd", "kind": "st", "nodes": 96, "edges": 240, "K": 2,
         "level": 1, "rows": 2_250, "N": 131_072},
        # Crude Monte Carlo, the check and the fallback where no reference
        # states exist yet: every sample goes through the system function.
        {"name": "montecarlo", "task": "montecarlo", "kind": "st", "nodes": 119, "edges": 295,
         "K": 2, "level": 1, "N": 1_000_000},
        # Exact match counts of every row: the violation-matrix form, against
        # rows that are no system's reference sets.
        {"name": "count_rows", "task": "count", "kind": "rows", "edges": 295, "K": 2,
         "rows": 100_000, "N": 1_000_000},
        # Many hazard scenarios of several networks in one captured graph.
        {"name": "plan_hazards", "task": "plan", "kind": "st", "nodes": 96, "edges": 240, "K": 2,
         "level": 1, "rows": 2_250, "graphs": 3, "scenarios": 16, "N": 65_536},
        # Growing reference sets from nothing.
        {"name": "stage1", "task": "stage1", "kind": "st", "nodes": 119, "edges": 295, "K": 2,
         "level": 1, "rows": 6_000, "picks": 1024, "N": 100_000},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# Networks of the batched study, smallest to largest, and the two graphs of
# the paper's sizes.
_NETS = ((12, 20), (50, 120), (69, 172), (96, 240), (134, 335), (186, 465), (259, 647),
         (360, 900), (500, 1250), (59, 262), (119, 295))


def draw(rng):
    """A case of the same ranges: sizes spread over their logarithms, odd ones
    among them; never dearer than the largest listed case."""
    task = rng.choice(("stage2",) * 7 + ("autograd", "autograd", "montecarlo", "count", "plan",
                                         "stage1"))
    nodes, edges = rng.choice(_NETS)
    if task == "count":
        c = {"task": task, "kind": "rows", "edges": rng.choice((172, 240, 295, 465)),
             "K": rng.choice((2, 2, 3)), "rows": _log_int(rng, 500, 50_000),
             "N": _log_int(rng, 20_000, 400_000)}
    elif task == "plan":
        nodes, edges = rng.choice(_NETS[1:6])
        c = {"task": task, "kind": "st", "nodes": nodes, "edges": edges, "K": rng.choice((2, 2, 3)),
             "level": 1, "rows": _log_int(rng, 200, 4_000), "graphs": rng.choice((1, 2, 3)),
             "scenarios": rng.choice((2, 5, 8, 16)), "N": _log_int(rng, 4_000, 65_536)}
    elif task == "stage1":
        nodes, edges = rng.choice(_NETS[1:5])
        c = {"task": task, "kind": rng.choice(("st", "st", "global")), "nodes": nodes,
             "edges": edges, "K": 2, "level": 1, "rows": _log_int(rng, 300, 6_000),
             "picks": _log_int(rng, 64, 1024), "N": _log_int(rng, 10_000, 100_000)}
    elif task == "montecarlo":
        nodes, edges = rng.choice(_NETS[1:8])
        c = {"task": task, "kind": "st", "nodes": nodes, "edges": edges, "K": 2, "level": 1,
             "N": _log_int(rng, 10_000, 400_000)}
    elif task == "autograd":
        nodes, edges = rng.choice(_NETS[:7])
        c = {"task": task, "kind": "st", "nodes": nodes, "edges": edges, "K": 2, "level": 1,
             "rows": _log_int(rng, 50, 10_000), "N": _log_int(rng, 5_000, 300_000)}
    else:
        kind = rng.choice(("st", "st", "st", "st", "global", "flow"))
        if kind == "st":
            K = rng.choice((2, 2, 2, 3))
            if K == 3 and edges > 647:
                nodes, edges = 119, 295
            level = rng.randint(1, K - 1)
            cap = 40_000 if edges >= 295 else 10_000
            c = {"task": task, "kind": kind, "nodes": nodes, "edges": edges, "K": K,
                 "level": level, "rows": _log_int(rng, 50, cap), "N": _log_int(rng, 5_000, 1_000_000)}
            if edges > 500 or K == 3:
                c["N"] = _log_int(rng, 5_000, 262_144)
        else:
            nodes, edges = rng.choice(((50, 120), (69, 172), (96, 240), (59, 262), (119, 295)))
            c = {"task": task, "kind": kind, "nodes": nodes, "edges": edges,
                 "K": 3 if kind == "flow" else 2,
                 "level": rng.randint(1, 2) if kind == "global" else rng.randint(2, 3),
                 "rows": _log_int(rng, 200, 4_000), "N": _log_int(rng, 5_000, 262_144)}
    if rng.random() < 0.4:
        c["N"] |= 1  # an odd count
    return c


# ---- inputs ---------------------------------------------------------------------


@functools.lru_cache(maxsize=None)
def _context():
    """One context per process, as a program on one GPU keeps."""
    return R.Context(0)


@functools.lru_cache(maxsize=None)
def _network(nodes, edges, variant=0):
    """A connected random geometric graph: each node joined to its nearest
    predecessor, then the closest other pairs, edges by increasing length.
    Source = the node of highest degree, sink = the most hops away."""
    rng = np.random.default_rng(9_000 + 31 * nodes + edges + 7 * variant)
    pos = rng.random((nodes, 2))
    iu, ju = np.triu_indices(nodes, k=1)
    d = np.hypot(pos[iu, 0] - pos[ju, 0], pos[iu, 1] - pos[ju, 1])
    full = np.full((nodes, nodes), np.inf)
    full[iu, ju] = full[ju, iu] = d
    near = [int(np.argmin(full[v, :v])) for v in range(1, nodes)]
    chosen = {(min(u, v), max(u, v)) for v, u in zip(range(1, nodes), near)}
    for k in np.argsort(d, kind="stable"):
        if len(chosen) >= edges:
            break
        chosen.add((int(iu[k]), int(ju[k])))
    pairs = np.array(sorted(chosen, key=lambda e: full[e[0], e[1]]), dtype=np.int32)
    eu, ev = np.ascontiguousarray(pairs[:, 0]), np.ascontiguousarray(pairs[:, 1])
    deg = np.bincount(np.concatenate([eu, ev]), minlength=nodes)
    source = int(np.argmax(deg))
    hops = np.full(nodes, nodes)
    hops[source] = 0
    for _ in range(nodes):
        before = hops.copy()
        np.minimum.at(hops, ev, before[eu] + 1)
        np.minimum.at(hops, eu, before[ev] + 1)
        if np.array_equal(before, hops):
            break
    return {"n_nodes": nodes, "edge_u": eu, "edge_v": ev, "source": source,
            "sink": int(np.argmax(hops))}


def _nominal_failure(edges):
    return np.random.default_rng(77 + edges).uniform(0.01, 0.20, edges)


def _shortest_trees(adj_node, adj_edge, root, w):
    """Shortest-path distances and predecessor slots from `root` under each
    row of w ([draws, edges + 1], the last column infinite padding)."""
    draws, nodes = w.shape[0], adj_node.shape[0]
    cost = w[:, adj_edge]
    dist = torch.full((draws, nodes), math.inf, device=w.device)
    dist[:, root] = 0.0
    pred = torch.zeros((draws, nodes), dtype=torch.int64, device=w.device)
    for _ in range(nodes):
        best, slot = (dist[:, adj_node] + cost).min(dim=2)
        closer = best < dist
        if not bool(closer.any()):
            break
        dist = torch.where(closer, best, dist)
        pred = torch.where(closer, slot, pred)
    return dist, pred


@functools.lru_cache(maxsize=None)
def _st_pool(nodes, edges, variant, rows):
    """About 1.25 * rows distinct s-t path sets and as many cut sets, as 0/1
    membership rows: shortest paths under randomly scaled weights, and the
    minimal cuts at the edge of a ball around either terminal."""
    g = _network(nodes, edges, variant)
    dev = torch.device("cuda")
    incident = [[] for _ in range(nodes)]
    for e, (u, v) in enumerate(zip(g["edge_u"].tolist(), g["edge_v"].tolist())):
        incident[u].append((v, e))
        incident[v].append((u, e))
    width = max(map(len, incident))
    adj = np.zeros((nodes, width, 2), dtype=np.int64)
    adj[:, :, 1] = edges
    for v, ne in enumerate(incident):
        adj[v, :len(ne)] = ne
    adj_node = torch.from_numpy(adj[:, :, 0].copy()).to(dev)
    adj_edge = torch.from_numpy(adj[:, :, 1].copy()).to(dev)
    eu = torch.from_numpy(g["edge_u"].astype(np.int64)).to(dev)
    ev = torch.from_numpy(g["edge_v"].astype(np.int64)).to(dev)
    want = rows + rows // 4
    rng = np.random.default_rng(1_000 * nodes + edges + variant)
    base = -np.log(1.0 - _nominal_failure(edges)) + 0.02
    paths, cuts = np.zeros((0, edges), np.uint8), np.zeros((0, edges), np.uint8)

    def distinct(a):
        keys = np.packbits(a, axis=1)
        _, first = np.unique(keys.view([("", keys.dtype)] * keys.shape[1]).ravel(),
                             return_index=True)
        return a[np.sort(first)]

    draws = int(min(8192, max(512, want // 3)))
    for attempt in range(16):
        # The noise grows: the most probable paths first, then the detours
        # that samples with several failures need.
        noise = rng.exponential(1.0, (draws, edges)) ** (1.0 + 0.5 * attempt)
        w = np.full((draws, edges + 1), np.inf, dtype=np.float32)
        w[:, :edges] = base * noise + 1e-6
        wt = torch.from_numpy(w).to(dev)
        s, t = g["source"], g["sink"]
        dist_s, pred = _shortest_trees(adj_node, adj_edge, s, wt)
        dist_t, _ = _shortest_trees(adj_node, adj_edge, t, wt)
        at = torch.full((draws,), t, dtype=torch.int64, device=dev)
        row = torch.zeros((draws, edges + 1), dtype=torch.uint8, device=dev)
        for _ in range(nodes):
            slot = pred.gather(1, at[:, None])[:, 0]
            e = torch.where(at == s, edges, adj_edge[at, slot])
            row.scatter_(1, e[:, None], 1)
            at = torch.where(at == s, at, adj_node[at, slot])
            if bool((at == s).all()):
                break
        paths = distinct(np.concatenate([paths, row[:, :edges].cpu().numpy()]))
        balls = []
        for dist, far in ((dist_t, s), (dist_s, t)):
            r = torch.from_numpy(rng.random(draws).astype(np.float32)).to(dev) * dist[:, far]
            inside = dist < torch.minimum(r + 1e-7, dist[:, far])[:, None]
            inside[:, far] = False
            inside[:, t if far == s else s] = True
            # The far terminal's component outside the ball: the edges into it
            # are a minimal cut.
            side = torch.zeros_like(inside)
            side[:, far] = True
            while True:
                wider = side | (side[:, adj_node] & (adj_edge < edges)).any(dim=2) & ~inside
                if bool((wider == side).all()):
                    break
                side = wider
            balls.append((side[:, eu] != side[:, ev]).to(torch.uint8))
        cuts = distinct(np.concatenate([cuts] + [b.cpu().numpy() for b in balls]))
        if len(paths) >= want and len(cuts) >= want:
            break
    return paths[:want], cuts[:want]


def _rows(case, rng, variant=0):
    """Reference rows (lower, upper) of an s-t system for the case's level."""
    K, level, rows = case["K"], case["level"], case["rows"]
    paths, cuts = _st_pool(case["nodes"], case["edges"], variant, rows)
    pick_p = rng.permutation(len(paths))[:rows]
    pick_c = rng.permutation(len(cuts))[:rows]
    upper = paths[pick_p] * np.uint8(level)
    lower = np.where(cuts[pick_c] > 0, level - 1, K - 1).astype(np.uint8)
    return lower, upper


def _probabilities(case, rng):
    """A hazard scenario: state probabilities [n][K] around the network's
    nominal ones."""
    n, K = case["edges"], case["K"]
    if case["kind"] == "rows":
        up = rng.uniform(0.7, 0.99, n)
        p = np.stack([1.0 - up, up], axis=1) if K == 2 else rng.dirichlet([1.0, 2.0, 8.0], size=n)
    elif K == 2:
        fail = np.clip(_nominal_failure(n) * np.exp(rng.normal(0.0, 0.25, n)), 1e-4, 0.5)
        p = np.stack([1.0 - (1.0 - fail), 1.0 - fail], axis=1)
    else:
        p = rng.dirichlet([8.0, 2.0, 1.0][:K], size=n)[:, ::-1].copy()
    return np.ascontiguousarray(p)


def prepare(case, seed):
    ctx = _context()
    rng = np.random.default_rng(seed)
    task, K, N = case["task"], case["K"], case["N"]
    st = {"case": case, "ctx": ctx, "N": N, "key": int(rng.integers(1, 1 << 40))}
    if task == "plan":
        st["keep"], jobs = [], []
        for variant in range(case["graphs"]):
            lower, upper = _rows(case, rng, variant)
            refs = R.Refs(ctx, case["edges"], K, lower, upper)
            system = R.System(ctx, _network(case["nodes"], case["edges"], variant), K=K,
                              level=case["level"], kind="st")
            for _ in range(case["scenarios"]):
                model = R.Model(ctx, _probabilities(case, rng))
                jobs.append({"model": model, "refs": refs, "system": system, "N": N,
                             "seed": st["key"] + len(jobs),
                             "buffers": R.Buffers(ctx, case["edges"], K, N)})
        st["jobs"] = jobs
        st["plan"] = R.Plan(ctx, jobs, tune=False)
        return st
    p = _probabilities(case, rng)
    st["model"] = R.Model(ctx, p)
    if task == "count":
        n, rows = case["edges"], case["rows"]
        lower = np.where(rng.random((rows, n), dtype=np.float32) < 0.9, K - 1, 0).astype(np.uint8)
        upper = np.where(rng.random((rows, n), dtype=np.float32) < 0.05, K - 1, 0).astype(np.uint8)
        st["refs"] = R.Refs(ctx, n, K, lower, upper)
        st["samples"] = R.rsr_sample(ctx, st["model"], st["key"], 0, 0, N)
        st["flags"] = torch.empty(N, dtype=torch.uint8, device=ctx.device)
        st["match"] = torch.empty((N, 2), dtype=torch.int32, device=ctx.device)
        return st
    st["system"] = R.System(ctx, _network(case["nodes"], case["edges"]), K=K, level=case["level"],
                            kind=case["kind"])
    if task == "stage1":
        st["rows"] = np.zeros((case["rows"], case["edges"]), dtype=np.uint8)
        return st
    st["buffers"] = R.Buffers(ctx, case["edges"], K, N)
    if task == "montecarlo":
        st["importance"] = torch.empty(case["edges"], dtype=torch.float32, device=ctx.device)
        return st
    if case["kind"] == "st":
        lower, upper = _rows(case, rng)
    else:
        lower, upper, _ = R.stage1(ctx, st["model"], st["system"], 20_000, 2048, 1e-3,
                                   case["rows"], 40, st["key"] + 1)
    st["refs"] = R.Refs(ctx, case["edges"], K, lower, upper)
    if task == "autograd":
        st["p"] = torch.from_numpy(p[:, 1].copy()).to(ctx.device).requires_grad_(True)
    return st


# ---- one pass --------------------------------------------------------------------


def run(st):
    case, ctx, N = st["case"], st["ctx"], st["N"]
    task = case["task"]
    if task == "stage2":
        est, b = R.stage2(ctx, st["model"], st["refs"], st["system"], N, st["key"],
                          buffers=st["buffers"])
        return {"estimate": est, "samples": b.samples, "flags": b.flags, "Y": b.Y, "G": b.G,
                "evaluated": b.n_eval}
    if task == "autograd":
        P = R.rsr_probability(st["p"], st["refs"], st["system"], N, st["key"], ctx)
        (grad,) = torch.autograd.grad(P, st["p"])
        return {"P": P, "grad": grad}
    if task == "montecarlo":
        b = st["buffers"]
        R.rsr_sample(ctx, st["model"], st["key"], 0, 0, N, out=b.samples)
        R.rsr_eval_unknown(ctx, st["system"], b.samples, N, None, which=R.RSR_ALL, Y=b.Y)
        R.rsr_importance(ctx, st["model"], b.samples, b.Y, N, I=st["importance"])
        return {"samples": b.samples, "Y": b.Y, "importance": st["importance"]}
    if task == "count":
        R.rsr_classify(ctx, st["refs"], st["samples"], N, mode=R.RSR_COUNT, flags=st["flags"],
                       match=st["match"])
        return {"flags": st["flags"], "match": st["match"]}
    if task == "plan":
        st["plan"].run()
        ests, grads = st["plan"].results()
        return {"counts": np.array([[e[k] for k in ("n_L", "n_U", "n_u", "n_both", "n_u_up")]
                                    for e in ests], dtype=np.int64),
                "P": np.array([e["P"] for e in ests]), "se": np.array([e["se"] for e in ests]),
                "G": np.stack(grads)}
    lower, upper, res = R.stage1(ctx, st["model"], st["system"], N, case["picks"], 1e-3,
                                 case["rows"], 50, st["key"])
    # Both sides go to the program's own table, unused rows zero.
    rows, used = st["rows"], len(lower) + len(upper)
    rows[:len(lower)] = lower
    rows[len(lower):used] = upper
    rows[used:] = 0
    return {"rows": rows, "result": res}


def work(case):
    """Bytes: the rows and probabilities in, the samples written and, where a
    caller gets them, flags, Y, counts and gradients out.  Flops: one 32-bit
    operation per Philox product and round, ten rounds per eight components;
    counting adds one per 32 (sample, constrained component) pairs."""
    n, K, N = case["edges"], case["K"], case["N"]
    words = (K - 1) * ((n + 31) // 32)
    jobs = case.get("graphs", 1) * case.get("scenarios", 1)
    row_bytes = 2 * case.get("rows", 0) * words * 4 * case.get("graphs", 1)
    if case["task"] == "count":
        return {"bytes": N * (words * 4 + 9) + row_bytes,
                "flops": N * case["rows"] * n * 0.15 * (K - 1) / 32}
    return {"bytes": jobs * (N * (words * 4 + 2) + 12 * n * K) + row_bytes,
            "flops": jobs * N * 20.0 * ((n + 7) // 8)}


# ---- the same in 64 bits ------------------------------------------------------------


def _philox(c0, c1, c2, c3, key):
    mask = 0xFFFFFFFF
    k0, k1 = key & mask, key >> 32

    def product(a, b):
        # 32 x 32 -> (high, low) in int64 without overflow.
        p = (a & 0xFFFF) * b
        q = (a >> 16) * b
        low = (p + ((q & 0xFFFF) << 16))
        return ((q >> 16) + (low >> 32)) & mask, low & mask

    for _ in range(10):
        ah, al = product(0xD2511F53, c0)
        bh, bl = product(0xCD9E8D57, c2)
        c0, c1, c2, c3 = bh ^ c1 ^ k0, bl, ah ^ c3 ^ k1, al
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return c0, c1, c2, c3


def _states(p, key, N):
    """Component states [n][N] uint8 by the library's documented generator."""
    dev = torch.device("cuda")
    n, K = p.shape
    cum = np.zeros((n, K - 1))
    run_sum = np.zeros(n)
    for s in range(K - 1):
        run_sum = run_sum + p[:, s]
        cum[:, s] = np.minimum(np.floor(run_sum * 4294967296.0), 4294967296.0)
    h = torch.arange(N, dtype=torch.int64, device=dev)
    zero = torch.zeros_like(h)
    x = torch.zeros((n, N), dtype=torch.uint8, device=dev)
    for block in range((n + 7) // 8):
        hi = _philox(zero + block, h, zero, zero, key)
        lo = _philox(zero + (block | 0x80000000), h, zero, zero, key)
        for j in range(min(8, n - 8 * block)):
            shift = 16 * (j % 2)
            u = (((hi[j // 2] >> shift) & 0xFFFF) << 16) | ((lo[j // 2] >> shift) & 0xFFFF)
            for s in range(K - 1):
                x[8 * block + j] += (u >= int(cum[8 * block + j, s])).to(torch.uint8)
    return x


def _grow(marked, usable, ends):
    """Closure of marked [nodes][N] over the usable edges [edges][N]."""
    while True:
        before = int(marked.sum())
        for order in (range(len(ends)), range(len(ends) - 1, -1, -1)):
            for e in order:
                u, v = ends[e]
                both = (marked[u] | marked[v]) & usable[e]
                marked[u] |= both
                marked[v] |= both
        if int(marked.sum()) == before:
            return marked


def _phi(case, x, variant=0):
    """System function [N] bool of the states x [n][N]."""
    g = _network(case["nodes"], case["edges"], variant)
    ends = list(zip(g["edge_u"].tolist(), g["edge_v"].tolist()))
    N, level = x.shape[1], case["level"]

    def start(v):
        m = torch.zeros((case["nodes"], N), dtype=torch.bool, device=x.device)
        m[v] = True
        return m

    if case["kind"] == "st":
        return _grow(start(g["source"]), x >= level, ends)[g["sink"]]
    if case["kind"] == "global":
        up = x >= 1
        ok = _grow(start(0), up, ends).all(dim=0)
        if level == 2:
            for e in range(len(ends)):
                cut = up.clone()
                cut[e] = False
                ok &= _grow(start(0), cut, ends).all(dim=0)
        return ok
    cap = x.to(torch.int8)
    flow = torch.zeros_like(cap)
    done = torch.ones(N, dtype=torch.bool, device=x.device)
    eu = torch.from_numpy(g["edge_u"].astype(np.int64)).to(x.device)
    ev = torch.from_numpy(g["edge_v"].astype(np.int64)).to(x.device)
    col = torch.arange(N, device=x.device)
    for _ in range(level):  # one unit at a time
        mark = start(g["source"])
        parent = torch.zeros((case["nodes"], N), dtype=torch.int64, device=x.device)
        while True:
            before = int(mark.sum())
            for e, (u, v) in enumerate(ends):
                to_v = mark[u] & ~mark[v] & (cap[e] > flow[e])
                to_u = mark[v] & ~mark[u] & (cap[e] > -flow[e])
                parent[v] = torch.where(to_v, e, parent[v])
                parent[u] = torch.where(to_u, e, parent[u])
                mark[v] |= to_v
                mark[u] |= to_u
            if int(mark.sum()) == before:
                break
        found = mark[g["sink"]]
        done &= found
        at = torch.where(found, g["sink"], g["source"])
        while bool((at != g["source"]).any()):
            moving = at != g["source"]
            e = parent[at, col]
            forward = ev[e] == at
            step = torch.where(moving, torch.where(forward, 1, -1), 0).to(torch.int8)
            flow[e, col] += step
            at = torch.where(moving, torch.where(forward, eu[e], ev[e]), at)
    return done


def _gradient(p, x, Y):
    N = x.shape[1]
    counts = np.stack([((x == s) & Y).sum(dim=1).cpu().numpy() for s in range(p.shape[1])], axis=1)
    with np.errstate(divide="ignore", invalid="ignore"):
        return np.where(p > 0, counts / (N * p), 0.0)


def _estimate(Y):
    N = Y.numel()
    P = int(Y.sum()) / N
    return P, math.sqrt(P * (1 - P) / N), math.sqrt((1 - P) / (N * P)) if P > 0 else math.inf


def exact(case, seed):
    task, K, N = case["task"], case["K"], case["N"]
    if task in ("count", "stage1"):
        return None  # whole numbers, and fractions of whole numbers
    if case["kind"] == "global" and case["level"] == 2 and case["edges"] > 270:
        return None  # one closure per edge takes too long
    rng = np.random.default_rng(seed)
    key = int(rng.integers(1, 1 << 40))
    if task == "plan":
        P, se, G = [], [], []
        for variant in range(case["graphs"]):
            _rows(case, rng, variant)  # the same draws as prepare()
            for _ in range(case["scenarios"]):
                p = _probabilities(case, rng)
                x = _states(p, key + len(P), N)
                Y = _phi(case, x, variant)
                est = _estimate(Y)
                P.append(est[0])
                se.append(est[1])
                G.append(_gradient(p, x, Y))
        return {"counts": None, "P": np.array(P), "se": np.array(se), "G": np.stack(G)}
    p = _probabilities(case, rng)
    if task == "autograd":
        p = np.stack([1.0 - p[:, 1], p[:, 1]], axis=1)
        p = p / p.sum(axis=1, keepdims=True)
    x = _states(p, key, N)
    Y = _phi(case, x)
    P, se, cov = _estimate(Y)
    G = _gradient(p, x, Y)
    if task == "autograd":
        return {"P": P, "grad": G[:, 1] - G[:, 0]}
    if task == "montecarlo":
        return {"samples": None, "Y": None, "importance": G[:, 1] - G[:, 0]}
    return {"estimate": {"n_L": None, "n_U": None, "n_u": None, "n_both": None, "n_u_up": None,
                         "N": None, "p_L": None, "p_U": None, "p_u": None, "P": P, "se": se,
                         "cov": cov},
            "samples": None, "flags": None, "Y": None, "G": G, "evaluated": None}
