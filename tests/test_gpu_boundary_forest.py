"""The boundary search by spanning forests where it can go wrong: edge counts
around a multiple of 64, parallel edges and self-loops, paths and rings (long
hook chains, long branches to cut), nodes that no edge reaches, upper planes,
graphs whose forests fill the LDS with one or two waves a block, both sides.
Rows and sides are compared with the oracle, which evaluates the system
function at every step."""
import numpy as np
import pytest
import torch

import oracle
import paper_2604_17066_amd as R

pytestmark = pytest.mark.gpu


def _graph(name, rng):
    if name.startswith("multi"):     # tree, chords, parallel edges and self-loops
        m = int(name[5:])
        n = max(2, m // 3)
        eu = np.concatenate([np.arange(1, n), rng.integers(0, n, m - n + 1)])
        ev = np.concatenate([[int(rng.integers(0, v)) for v in range(1, n)],
                             rng.integers(0, n, m - n + 1)])
    elif name == "path":             # nodes in a shuffled order, every edge twice
        n = 70
        at = rng.permutation(n)
        eu, ev = np.concatenate([at[:-1], at[1:]]), np.concatenate([at[1:], at[:-1]])
        o = rng.permutation(eu.size)
        eu, ev = eu[o], ev[o]
    elif name == "ring":
        n = 129
        o = rng.permutation(n)
        eu, ev = o, (o + 1) % n
    elif name == "loose":            # nodes 20..29 have no edge
        n = 30
        eu, ev = rng.integers(0, 20, 60), rng.integers(0, 20, 60)
    else:                            # "wide<nodes>": few waves per block
        n = int(name[4:])
        m = 150
        eu, ev = rng.integers(0, 60, m), rng.integers(0, 60, m)
        eu[:2], ev[:2] = [59, 58], [n - 1, n - 2]
    return {"n_nodes": int(n), "edge_u": np.asarray(eu, np.int32), "edge_v": np.asarray(ev, np.int32),
            "source": 0, "sink": int(n) - 1}


@pytest.mark.parametrize("kind", ["st", "global"])
@pytest.mark.parametrize("name,K,level,up,picks", [
    ("multi1", 2, 1, 0.5, 64), ("multi63", 2, 1, 0.8, 200), ("multi64", 2, 1, 0.8, 200),
    ("multi65", 3, 2, 0.8, 200), ("multi257", 2, 1, 0.85, 101), ("path", 2, 1, 0.9, 120),
    ("ring", 2, 1, 0.985, 120), ("loose", 2, 1, 0.6, 90), ("wide1200", 2, 1, 0.8, 33),
    ("wide3000", 2, 1, 0.8, 33), ("wide4096", 2, 1, 0.8, 5)])
def test_rows_and_sides(rsr_ctx, kind, name, K, level, up, picks):
    if kind == "global":
        level = 1
        if name == "wide4096":
            pytest.skip("a graph that the search refuses for global connectivity")
    rng = np.random.default_rng([len(name), K, picks])
    graph = _graph(name, rng)
    n = graph["edge_u"].size
    p = np.empty((n, K))
    p[:, K - 1] = rng.uniform(up, 1.0, n)
    p[:, :K - 1] = ((1.0 - p[:, K - 1]) / (K - 1))[:, None]
    N = 256
    model = R.Model(rsr_ctx, p)
    xs = R.rsr_sample(rsr_ctx, model, 12, 0, 0, N)
    system = R.System(rsr_ctx, graph, K=K, level=level, kind=kind)
    pick = rng.choice(N, size=picks, replace=False).astype(np.int64)
    rows, side = R.rsr_boundary_search(rsr_ctx, system, xs, N,
                                       torch.tensor(pick, device=rsr_ctx.device))
    torch.cuda.synchronize()
    x = oracle.sample(p, 12, 0, 0, N)[pick]
    if kind == "global":
        want_rows, want_side, _ = oracle.boundary_global(graph, x, K=K, level=level)
    else:
        want_rows, want_side, _ = oracle.boundary_st(graph, x, K=K, level=level)
    print(kind, name, "upper picks:", int(want_side.sum()), "of", picks)
    np.testing.assert_array_equal(side.cpu().numpy(), want_side)
    np.testing.assert_array_equal(rows.cpu().numpy(), want_rows)
