"""The Stage-1 loop's row sets where they can go wrong: more rows than the
first table of distinct rows holds, many duplicates, given rows (equal ones
among them, and ones that contradict the system), both systems with a level.
Rows, their order and every count are compared with the oracle's loop."""
import numpy as np
import pytest

import oracle
import paper_2604_17066_amd as R
import workloads as WL

pytestmark = pytest.mark.gpu

KEYS = ("iterations", "p_u", "searches", "duplicates")


@pytest.mark.parametrize("kind,given,picks,iters,max_rows", [
    ("st", "none", 900, 3, 5_000), ("st", "equal", 40, 3, 5_000), ("st", "contradicting", 40, 2, 500),
    ("global", "none", 300, 2, 5_000), ("st", "none", 700, 4, 601)])
def test_rows_in_order(rsr_ctx, kind, given, picks, iters, max_rows):
    c = WL.configs.graph2(N=1, R_U=30, R_L=30)
    graph, p, N = c["graph"], c["p"], 6_000
    lower0 = upper0 = None
    if given == "equal":
        lower0, upper0 = np.repeat(c["lower"], 2, axis=0), np.concatenate([c["upper"], c["upper"]])
    elif given == "contradicting":     # upper rows below lower rows
        upper0 = c["upper"]
        lower0 = np.concatenate([c["lower"], c["upper"][:3] | c["lower"][:3]])
    model = R.Model(rsr_ctx, p)
    system = R.System(rsr_ctx, graph, kind=kind)
    lo, up, info = R.stage1(rsr_ctx, model, system, N, picks, 1e-9, max_rows, iters, 23,
                            lower0=lower0, upper0=upper0)
    wlo, wup, winfo = oracle.stage1(graph, p, N, picks, 1e-9, max_rows, iters, 23, lower0=lower0,
                                    upper0=upper0, kind=kind)
    print(kind, given, info)
    for key in KEYS:
        assert info[key] == winfo[key], key
    np.testing.assert_array_equal(lo, wlo)
    np.testing.assert_array_equal(up, wup)


def test_many_duplicates(rsr_ctx):
    c = WL.configs.tiny(N=10)
    graph, p = c["graph"], WL.configs.binary_model(c["p"][:, 1] * 0.9)
    model, system = R.Model(rsr_ctx, p), R.System(rsr_ctx, graph)
    lo, up, info = R.stage1(rsr_ctx, model, system, 5_000, 3_000, 1e-9, 10_000, 20, 4)
    wlo, wup, winfo = oracle.stage1(graph, p, 5_000, 3_000, 1e-9, 10_000, 20, 4)
    for key in KEYS:
        assert info[key] == winfo[key], key
    assert info["duplicates"] > 1_000
    np.testing.assert_array_equal(lo, wlo)
    np.testing.assert_array_equal(up, wup)


@pytest.mark.parametrize("picks", [2 ** 40, 2 ** 61, 2 ** 63 - 1])
def test_more_picks_than_samples(rsr_ctx, picks):
    """Room for the picks that a sample set can have, not for those asked for: seven
    components and 2^61 picks would come to a multiple of 2^64 bytes."""
    graph = {"n_nodes": 5, "edge_u": np.array([0, 0, 1, 1, 2, 3, 0]),
             "edge_v": np.array([1, 2, 2, 3, 4, 4, 3]), "source": 0, "sink": 4}
    p = np.tile([0.3, 0.7], (7, 1))
    model, system = R.Model(rsr_ctx, p), R.System(rsr_ctx, graph)
    lo, up, info = R.stage1(rsr_ctx, model, system, 500, picks, 1e-9, 1000, 5, 4)
    wlo, wup, winfo = oracle.stage1(graph, p, 500, 500, 1e-9, 1000, 5, 4)
    for key in KEYS:
        assert info[key] == winfo[key], key
    np.testing.assert_array_equal(lo, wlo)
    np.testing.assert_array_equal(up, wup)
