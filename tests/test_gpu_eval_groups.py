"""Evaluation of the system function 64 samples at a time, where it can go
wrong: ragged sample and edge counts, parallel edges and self-loops, graphs
made of ears (rings, chains of rings, ladders), the switch from a block to a
wave per group, graphs with few waves per block, upper planes, unaligned
flags, and the list of unclassified samples across its regions.  Everything is
compared with the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2604_17066_amd as R
from helpers import unpack_states

pytestmark = pytest.mark.gpu


def _graph(name, rng):
    if name == "ring":
        n = 23
        eu, ev = np.arange(n), (np.arange(n) + 1) % n
    elif name == "rings":        # rings joined at nodes, and one bridge in the middle
        eu, ev, at = [], [], 0
        for k, size in enumerate((3, 5, 2, 7, 4)):
            ring = [at] + list(range(at + 1, at + size))
            eu += ring
            ev += ring[1:] + [at]
            at += size - 1
            if k == 2:
                eu.append(at)
                ev.append(at + 1)
                at += 1
        n = at + 1
    elif name == "ladder":
        m = 20
        eu = list(range(m - 1)) + list(range(m, 2 * m - 1)) + list(range(m))
        ev = list(range(1, m)) + list(range(m + 1, 2 * m)) + list(range(m, 2 * m))
        n = 2 * m
    elif name == "multigraph":   # parallel edges, self-loops, 97 edges on 30 nodes
        n = 30
        eu = np.concatenate([np.arange(1, n), rng.integers(0, n, 68)])
        ev = np.concatenate([[int(rng.integers(0, v)) for v in range(1, n)], rng.integers(0, n, 68)])
    elif name == "pair":         # two nodes, two edges
        n, eu, ev = 2, [0, 1], [1, 0]
    else:                        # "large": few waves per block
        n, m = 900, 2400
        eu = np.concatenate([np.arange(1, n), rng.integers(0, n, m - n + 1)])
        ev = np.concatenate([[int(rng.integers(max(0, v - 9), v)) for v in range(1, n)],
                             rng.integers(0, n, m - n + 1)])
    return {"n_nodes": int(n), "edge_u": np.asarray(eu, np.int32), "edge_v": np.asarray(ev, np.int32),
            "source": 0, "sink": int(n) - 1}


CASES = [("ring", 2, 0.97, 1), ("ring", 3, 0.97, 63), ("rings", 2, 0.96, 4000),
         ("ladder", 2, 0.93, 4097), ("multigraph", 2, 0.9, 70_001), ("multigraph", 3, 0.9, 65),
         ("pair", 2, 0.6, 129), ("large", 2, 0.98, 400)]


@pytest.mark.parametrize("name,K,up,N", CASES)
def test_every_sample(rsr_ctx, name, K, up, N):
    rng = np.random.default_rng(N)
    g = _graph(name, rng)
    n = g["edge_u"].size
    p = np.full((n, K), (1 - up) / (K - 1))
    p[:, K - 1] = up
    model = R.Model(rsr_ctx, p)
    xs = R.rsr_sample(rsr_ctx, model, 8, 0, 0, N)
    x = unpack_states(xs.cpu().numpy(), n, K)
    for level in range(1, K):
        sys = R.System(rsr_ctx, g, K=K, level=level, kind="st")
        got = R.rsr_eval_unknown(rsr_ctx, sys, xs, N, None, which=R.RSR_ALL).cpu().numpy()
        want, _ = oracle.eval_unknown(g, x, None, which=1, level=level)
        np.testing.assert_array_equal(got, want, err_msg=f"st level {level}")
    for level in (1, 2):
        sys = R.System(rsr_ctx, g, K=K, level=level, kind="global")
        got = R.rsr_eval_unknown(rsr_ctx, sys, xs, N, None, which=R.RSR_ALL).cpu().numpy()
        want, _ = oracle.eval_unknown_global(g, x, None, which=1, level=level)
        np.testing.assert_array_equal(got, want, err_msg=f"global level {level}")


# Listed samples: none, few (a block per group), many (a wave per group), and
# more tiles of flags than regions (N > 512 * 1024).
@pytest.mark.parametrize("N,share,offset", [(1000, 0.0, 0), (1023, 0.05, 1), (4096, 1.0, 0),
                                            (70_003, 0.6, 3), (540_001, 0.02, 2)])
def test_listed_samples(rsr_ctx, N, share, offset):
    rng = np.random.default_rng(N)
    g = _graph("multigraph", rng)
    n = g["edge_u"].size
    model = R.Model(rsr_ctx, np.tile([[0.15, 0.85]], (n, 1)))
    xs = R.rsr_sample(rsr_ctx, model, 9, 0, 0, N)
    flags = np.where(rng.random(N) < share, 0, rng.integers(1, 4, N)).astype(np.uint8)
    d = torch.zeros(N + 8, dtype=torch.uint8, device=rsr_ctx.device)
    d[offset:offset + N] = torch.from_numpy(flags).to(rsr_ctx.device)
    out = torch.full((N + 8,), 77, dtype=torch.uint8, device=rsr_ctx.device)
    n_eval = torch.zeros(1, dtype=torch.int64, device=rsr_ctx.device)
    x = unpack_states(xs.cpu().numpy(), n, 2)
    for kind, ref in (("st", oracle.eval_unknown), ("global", oracle.eval_unknown_global)):
        sys = R.System(rsr_ctx, g, level=1, kind=kind)
        R.rsr_eval_unknown(rsr_ctx, sys, xs, N, d[offset:offset + N], Y=out[offset:offset + N],
                           n_evaluated=n_eval)
        got = out.cpu().numpy()
        want, _ = ref(g, x, flags)
        np.testing.assert_array_equal(got[offset:offset + N], want, err_msg=kind)
        assert (got[:offset] == 77).all() and (got[offset + N:] == 77).all()
        assert int(n_eval) == int((flags == 0).sum())


@pytest.mark.parametrize("n,m,up,N,seed", [
    (7, 12, 0.85, 5000, 7), (33, 80, 0.9, 20_000, 33), (50, 120, 0.9, 50_000, 50),
    (63, 150, 0.9, 20_000, 63), (64, 154, 0.9, 20_000, 66), (90, 216, 0.92, 20_000, 90),
    (150, 460, 0.9, 3000, 151), (200, 470, 0.93, 3000, 205)])
def test_two_edge_connectivity_of_local_graphs(rsr_ctx, n, m, up, N, seed):
    """Near neighbours joined, so that many samples have a single bridge or hang
    together by a few ears; lanes and waves without a node (fewer than 64, or not a
    multiple of 64) beside those that have one."""
    rng = np.random.default_rng(seed)
    pos = rng.random((n, 2))
    iu, ju = np.triu_indices(n, k=1)
    d = np.hypot(*(pos[iu] - pos[ju]).T)
    near = {(int(np.argmin(np.hypot(*(pos[:v] - pos[v]).T))), v) for v in range(1, n)}
    for v in range(n):  # and two neighbours at least
        near |= {(min(int(w), v), max(int(w), v))
                 for w in np.argsort(np.hypot(*(pos - pos[v]).T))[1:3]}
    for k in np.argsort(d, kind="stable"):
        if len(near) >= m:
            break
        near.add((int(iu[k]), int(ju[k])))
    ends = np.array(sorted(near, key=lambda e: float(np.hypot(*(pos[e[0]] - pos[e[1]])))), np.int32)
    g = {"n_nodes": n, "edge_u": ends[:, 0].copy(), "edge_v": ends[:, 1].copy(), "source": 0,
         "sink": n - 1}
    system = R.System(rsr_ctx, g, kind="global", level=2)
    # Two thirds of the edges are sure, so that the rest decide.
    q = np.where(rng.random(len(ends)) < 0.6, 1.0 - (1.0 - up) / 20, up)
    model = R.Model(rsr_ctx, np.stack([1.0 - q, q], axis=1))
    xs = R.rsr_sample(rsr_ctx, model, 7, 0, 0, N)
    x = unpack_states(xs.cpu().numpy(), len(ends), 2)
    want, _ = oracle.eval_unknown_global(g, x, None, which=1, level=2)
    assert 0 < want.sum() < N
    Y = R.rsr_eval_unknown(rsr_ctx, system, xs, N, None, which=R.RSR_ALL)
    np.testing.assert_array_equal(Y.cpu().numpy(), want)
    # The same samples listed, in groups of others.
    flags = torch.from_numpy((rng.random(N) < 0.4).astype(np.uint8)).to(rsr_ctx.device)
    Y = R.rsr_eval_unknown(rsr_ctx, system, xs, N, flags).cpu().numpy()
    open_ = flags.cpu().numpy() == 0
    np.testing.assert_array_equal(Y[open_], want[open_])


def test_large_tables_keep_a_block_busy(rsr_ctx):
    """A few samples on a graph whose tables leave a block room for one group: its
    waves share the sweeps, so four times the edges of a graph with room for four
    groups take about a quarter more, not three times as long."""
    rng = np.random.default_rng(5)
    us = []
    for m in (1000, 4000):
        eu = np.concatenate([np.arange(99), rng.integers(0, 100, m - 99)]).astype(np.int32)
        ev = np.concatenate([np.arange(1, 100), rng.integers(0, 100, m - 99)]).astype(np.int32)
        g = {"n_nodes": 100, "edge_u": eu, "edge_v": ev, "source": 0, "sink": 99}
        system = R.System(rsr_ctx, g)
        model = R.Model(rsr_ctx, np.tile([0.7, 0.3], (m, 1)))
        xs = R.rsr_sample(rsr_ctx, model, 7, 0, 0, 20)
        Y = R.rsr_eval_unknown(rsr_ctx, system, xs, 20, None, which=R.RSR_ALL)
        x = unpack_states(xs.cpu().numpy(), m, 2)
        np.testing.assert_array_equal(Y.cpu().numpy(), oracle.eval_unknown(g, x, None, which=1)[0])
        best = float("inf")
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(50):
                R.rsr_eval_unknown(rsr_ctx, system, xs, 20, None, which=R.RSR_ALL, Y=Y)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) * 20)
        us.append(best)
    assert us[1] < 2 * us[0], us


def _cliques(count, size):
    """A chain of cliques, two links between neighbours: an ear for every link."""
    e = []
    for k in range(count):
        e += [(size * k + a, size * k + b) for a in range(size) for b in range(a + 1, size)]
        if k:
            e += [(size * (k - 1), size * k), (size * (k - 1) + 1, size * k + 1)]
    return size * count, e


def _roads(side, pieces):
    """A lattice of crossings whose roads are chains of `pieces` edges."""
    n, e = side * side, []
    for a, b in ([(r * side + c, r * side + c + 1) for r in range(side) for c in range(side - 1)] +
                 [(r * side + c, r * side + c + side) for r in range(side - 1) for c in range(side)]):
        for _ in range(pieces - 1):
            e.append((a, n))
            a, n = n, n + 1
        e.append((a, b))
    return n, e


def _ladder(m):
    return 2 * m, ([(i, i + 1) for i in range(m - 1)] + [(m + i, m + i + 1) for i in range(m - 1)] +
                   [(i, m + i) for i in range(m)])


def _dense(n, m, rng):
    return n, [(i, i + 1) for i in range(n - 1)] + rng.integers(0, n, (m - n + 1, 2)).tolist()


# More samples than the walk's waves take at once (8192), so that the search of 64
# goes first, with ears or without, and leaves some; few samples on a shallow
# graph, which it takes too, and on others, which go to the walk; tables just
# within the LDS and beyond it.
@pytest.mark.parametrize("name,up,N", [
    ("ladder", 0.99, 9001), ("roads", 0.996, 8300), ("cliques", 0.97, 8193),
    ("short cliques", 0.9, 20_000), ("shallow", 0.85, 700), ("deep", 0.999, 300),
    ("tables fit", 0.2, 130), ("tables too large", 0.2, 130)])
def test_two_edge_connectivity_by_search_and_walk(rsr_ctx, name, up, N):
    rng = np.random.default_rng(len(name))
    n, e = {"ladder": lambda: _ladder(60), "roads": lambda: _roads(7, 3),
            "cliques": lambda: _cliques(40, 8), "short cliques": lambda: _cliques(5, 8),
            "shallow": lambda: _dense(120, 300, rng), "deep": lambda: _ladder(130),
            "tables fit": lambda: _dense(200, 4000, rng),
            "tables too large": lambda: _dense(200, 4096, rng)}[name]()
    ends = np.array(e, np.int32)
    g = {"n_nodes": n, "edge_u": ends[:, 0].copy(), "edge_v": ends[:, 1].copy(), "source": 0,
         "sink": n - 1}
    system = R.System(rsr_ctx, g, kind="global", level=2)
    if name == "shallow":  # the first edges are the only path to the ends
        up = np.where(np.bincount(ends.ravel(), minlength=n)[ends].min(axis=1) < 4, 0.995, up)
    q = np.broadcast_to(up, len(e)).astype(np.float64)
    model = R.Model(rsr_ctx, np.stack([1.0 - q, q], axis=1))
    xs = R.rsr_sample(rsr_ctx, model, 7, 0, 0, N)
    # The oracle on the first samples; the others in parts of 4000, which the walk
    # takes alone (but on shallow graphs).
    some = min(N, 130 if len(e) < 1000 else 6)
    x = unpack_states(xs[:, :some].cpu().numpy(), len(e), 2)
    first, _ = oracle.eval_unknown_global(g, x, None, which=1, level=2)
    want = np.concatenate([
        R.rsr_eval_unknown(rsr_ctx, system, R.rsr_sample(rsr_ctx, model, 7, 0, at, part), part, None,
                           which=R.RSR_ALL).cpu().numpy()
        for at in range(0, N, 4000) for part in [min(4000, N - at)]])
    np.testing.assert_array_equal(want[:some], first)
    n_eval = torch.zeros(1, dtype=torch.int64, device=rsr_ctx.device)
    Y = R.rsr_eval_unknown(rsr_ctx, system, xs, N, None, which=R.RSR_ALL, n_evaluated=n_eval)
    np.testing.assert_array_equal(Y.cpu().numpy(), want)
    assert int(n_eval) == N
    assert name == "shallow" or 0 < want.sum() < N
    flags = torch.from_numpy((rng.random(N) < 0.05).astype(np.uint8)).to(rsr_ctx.device)
    open_ = flags.cpu().numpy() == 0
    Y = R.rsr_eval_unknown(rsr_ctx, system, xs, N, flags, n_evaluated=n_eval)
    np.testing.assert_array_equal(Y.cpu().numpy(), np.where(open_, want, 0))
    assert int(n_eval) == open_.sum()


def test_two_edge_connectivity_in_a_plan(rsr_ctx):
    """Jobs of different sizes share the search and the walk."""
    n, e = _roads(5, 2)
    ends = np.array(e, np.int32)
    g = {"n_nodes": n, "edge_u": ends[:, 0].copy(), "edge_v": ends[:, 1].copy(), "source": 0,
         "sink": n - 1}
    m = len(e)
    system = R.System(rsr_ctx, g, kind="global", level=2)
    lower = np.ones((m, m), np.uint8) - np.eye(m, dtype=np.uint8)
    refs = R.Refs(rsr_ctx, m, 2, lower[:9], np.ones((1, m), np.uint8))
    model = R.Model(rsr_ctx, np.tile([0.02, 0.98], (m, 1)))
    jobs = [{"model": model, "refs": refs, "system": system, "seed": 70 + k, "N": N,
             "buffers": R.Buffers(rsr_ctx, m, 2, N)} for k, N in enumerate((5000, 77, 3201))]
    plan = R.Plan(rsr_ctx, jobs, tune=False)
    plan.run()
    plan.results()
    want = []
    for job in jobs:
        x = unpack_states(job["buffers"].samples.cpu().numpy(), m, 2)
        want.append(oracle.eval_unknown_global(g, x, None, which=1, level=2)[0])
        np.testing.assert_array_equal(job["buffers"].Y.cpu().numpy(), want[-1])
        job["buffers"].Y.fill_(9)
    plan.run()
    plan.results()
    for job, Y in zip(jobs, want):
        np.testing.assert_array_equal(job["buffers"].Y.cpu().numpy(), Y)
    plan.close()


def test_many_ears_do_not_take_forever(rsr_ctx):
    """A ladder has an ear per rung: two-edge-connectivity takes a few times as long
    as connectivity, not as many times as there are rungs."""
    n, e = _ladder(500)
    ends = np.array(e, np.int32)
    g = {"n_nodes": n, "edge_u": ends[:, 0].copy(), "edge_v": ends[:, 1].copy(), "source": 0,
         "sink": n - 1}
    model = R.Model(rsr_ctx, np.tile([0.01, 0.99], (len(e), 1)))
    ms = []
    for level in (1, 2):
        system = R.System(rsr_ctx, g, kind="global", level=level)
        xs = R.rsr_sample(rsr_ctx, model, 7, 0, 0, 300)
        Y = R.rsr_eval_unknown(rsr_ctx, system, xs, 300, None, which=R.RSR_ALL)
        best = float("inf")
        for _ in range(3):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            R.rsr_eval_unknown(rsr_ctx, system, xs, 300, None, which=R.RSR_ALL, Y=Y)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        ms.append(best)
    assert ms[1] < 15 * ms[0], ms
