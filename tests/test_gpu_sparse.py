"""The sparse LABEL form (the automatic one on consistent rows that constrain
few components) where it can go wrong: tile, slice and round boundaries, ragged
widths, more tiles than blocks, empty sides, unaligned flags and jobs of a
plan whose sizes differ.  Small cases against the oracle, large ones against
the popcount form."""
import time

import numpy as np
import pytest
import torch

import oracle
import paper_2604_17066_amd as R
from helpers import unpack_states

pytestmark = pytest.mark.gpu


def _rows(rng, R_L, R_U, n, K, bits):
    """Consistent rows: component 0 is 0 in every lower and K-1 in every upper
    row; about `bits` further components are constrained, in rows of mixed
    sizes."""
    lower = np.full((R_L, n), K - 1, dtype=np.uint8)
    upper = np.zeros((R_U, n), dtype=np.uint8)
    for rows, at, far in ((lower, 0, K - 1), (upper, K - 1, 0)):
        share = rng.uniform(0.3, 2.0, rows.shape[0])[:, None] * bits / n
        hit = rng.random(rows.shape) < share
        level = rng.integers(0, K, rows.shape).astype(np.uint8)
        rows[hit] = level[hit]
        rows[:, 0] = at
    return lower, upper


def _model(n, K, bits):
    q = max(0.5, 1.0 - 3.0 / bits)
    p = np.full((n, K), (1.0 - q) / (K - 1))
    p[:, K - 1] = 1.0 - (1.0 - q) / (K - 1) * (K - 1)
    p[0] = 1.0 / K
    return p


def _flags(ctx, model, refs, seed, N, form=R.RSR_AUTO, offset=0):
    xs = R.rsr_sample(ctx, model, seed, 0, 0, N)
    out = torch.full((N + offset + 8,), 77, dtype=torch.uint8, device=ctx.device)
    R.rsr_classify(ctx, refs, xs, N, form=form, flags=out[offset:offset + N])
    got = out.cpu().numpy()
    assert (got[:offset] == 77).all() and (got[offset + N:] == 77).all()
    return xs, got[offset:offset + N]


@pytest.mark.parametrize("n,K,R_L,R_U,N,offset", [
    (5, 2, 1, 1, 1, 0),
    (31, 2, 63, 64, 127, 0),
    (32, 2, 64, 65, 128, 0),
    (33, 2, 65, 300, 129, 3),
    (70, 3, 255, 257, 4097, 1),
    (40, 4, 384, 385, 2047, 2),
    (64, 2, 700, 9, 10_001, 0),
    (295, 2, 0, 500, 3000, 0),
    (295, 2, 500, 0, 3001, 0),
    (295, 2, 1500, 4500, 6000, 5),
    (1250, 2, 400, 450, 2500, 0),
    (21, 16, 300, 330, 3000, 0),
])
def test_small_against_the_oracle(rsr_ctx, n, K, R_L, R_U, N, offset):
    rng = np.random.default_rng(n * 31 + N)
    bits = min(12, max(1, n // 3))
    lower, upper = _rows(rng, R_L, R_U, n, K, bits)
    model = R.Model(rsr_ctx, _model(n, K, bits))
    refs = R.Refs(rsr_ctx, n, K, lower, upper)
    assert refs.consistent
    xs, got = _flags(rsr_ctx, model, refs, 11, N, offset=offset)
    want, _, _ = oracle.classify(lower, upper, unpack_states(xs.cpu().numpy(), n, K), mode=0)
    np.testing.assert_array_equal(got, want)
    if N > 2000 and R_L and R_U:
        assert {1, 2} <= set(np.unique(got).tolist())


# More tiles than blocks (512 of them): tiles of 2048 samples up to about 300
# bits, of 512 at 1250, of 128 at 4096; three rounds from 6145 rows on.
@pytest.mark.parametrize("n,K,R_L,R_U,N", [
    (60, 2, 900, 7000, 1_100_001),
    (295, 2, 7000, 400, 1_050_000),
    (1250, 2, 900, 900, 270_003),
    (4096, 2, 300, 500, 66_001),
    (295, 3, 20, 20, 600_001),
])
def test_large_against_the_popcount_form(rsr_ctx, n, K, R_L, R_U, N):
    rng = np.random.default_rng(n + N)
    lower, upper = _rows(rng, R_L, R_U, n, K, 14)
    model = R.Model(rsr_ctx, _model(n, K, 14))
    refs = R.Refs(rsr_ctx, n, K, lower, upper)
    assert refs.consistent
    _, got = _flags(rsr_ctx, model, refs, 12, N)
    _, want = _flags(rsr_ctx, model, refs, 12, N, form=R.RSR_POPCOUNT)
    np.testing.assert_array_equal(got, want)
    assert {1, 2} <= set(np.unique(got).tolist())


@pytest.mark.parametrize("n,K,upper_side", [(5, 2, True), (7, 2, True), (8, 2, False), (15, 2, True),
                                            (4, 3, True), (5, 4, False)])
def test_few_bits_many_undecided(rsr_ctx, n, K, upper_side):
    """A list of survivors that takes more room than the columns of its tile: fewer
    than 16 bits, three rounds (more than 6144 rows), more undecided samples
    (524288) than the smaller tiles hold, some of them decided in the last
    round."""
    N, top = 1_100_003, K - 1
    first, later = [0, 1], [0, 2, 3]
    if n >= 8:
        first, later = [0, 1, 2], [0, 3, 4, 5]
    far, near = (top, 0) if upper_side else (0, top)
    rows = np.full((7000, n), near, dtype=np.uint8)
    rows[:6200, first] = far
    rows[6200:, later] = far
    none = np.zeros((0, n), dtype=np.uint8)
    refs = R.Refs(rsr_ctx, n, K, *((none, rows) if upper_side else (rows, none)))
    p = np.full((n, K), 0.12)
    p[:, near] = 0.0
    p[:, near] = 1.0 - p.sum(axis=1)
    model = R.Model(rsr_ctx, p)
    xs, got = _flags(rsr_ctx, model, refs, 13, N)
    x = unpack_states(xs.cpu().numpy(), n, K)

    def hit(row):
        return (x >= row).all(axis=1) if upper_side else (x <= row).all(axis=1)

    early, late = hit(rows[0]), hit(rows[6200])
    assert (~early).sum() > 600_000 and (late & ~early).sum() > 100
    np.testing.assert_array_equal(got, np.where(early | late, 2 if upper_side else 1, 0))


def test_rows_without_a_bit_and_dense_rows_keep_their_labels(rsr_ctx):
    rng = np.random.default_rng(3)
    n, N = 40, 5000
    model = R.Model(rsr_ctx, np.full((n, 2), 0.5))
    dense = rng.random((300, n)) < 0.9
    for lower, upper in ((np.ones((2, n), np.uint8), np.zeros((0, n), np.uint8)),
                         (np.zeros((0, n), np.uint8), np.zeros((3, n), np.uint8)),
                         (np.zeros((0, n), np.uint8), dense.astype(np.uint8))):
        refs = R.Refs(rsr_ctx, n, 2, lower, upper)
        xs, got = _flags(rsr_ctx, model, refs, 4, N)
        want, _, _ = oracle.classify(lower, upper, unpack_states(xs.cpu().numpy(), n, 2), mode=0)
        np.testing.assert_array_equal(got, want)


@pytest.mark.parametrize("sizes", [(1, 127, 128, 129), (5000, 3, 2048, 70_001, 64),
                                   tuple([4099] * 40)])
def test_jobs_of_a_plan(rsr_ctx, sizes):
    """Jobs that end inside a tile, in one round and in the listed rounds."""
    n, K = 60, 3
    rng = np.random.default_rng(len(sizes))
    g = {"n_nodes": n + 1, "edge_u": np.arange(n), "edge_v": np.arange(1, n + 1), "source": 0,
         "sink": n}
    for rows in (50, 6500):
        lower, upper = _rows(rng, rows, rows, n, K, 12)
        refs = R.Refs(rsr_ctx, n, K, lower, upper)
        assert refs.consistent
        system = R.System(rsr_ctx, g, K=K, level=1)
        model = R.Model(rsr_ctx, _model(n, K, 12))
        jobs = [{"model": model, "refs": refs, "system": system, "seed": 50 + k, "N": N,
                 "buffers": R.Buffers(rsr_ctx, n, K, N)} for k, N in enumerate(sizes)]
        plan = R.Plan(rsr_ctx, jobs, tune=False)
        for _ in range(2):
            for job in jobs:
                job["buffers"].flags.fill_(9)
            plan.run()
            plan.results()
            for job in jobs:
                b = job["buffers"]
                want = R.rsr_classify(rsr_ctx, refs, b.samples, job["N"], form=R.RSR_POPCOUNT)
                np.testing.assert_array_equal(b.flags.cpu().numpy(), want.cpu().numpy())
        plan.close()


@pytest.mark.parametrize("sizes", [(200_001, 1, 2, 127, 128, 129, 3, 4097),
                                   tuple([50] * 129 + [700_000]), tuple([700_000] + [50] * 129),
                                   tuple([3] * 2100 + [400_000] + [130] * 2100)])
def test_jobs_of_very_different_sizes(rsr_ctx, sizes):
    """A block finds its job among up to 64, 64^2 and more; large jobs take more
    than one tile a block, small ones less than one."""
    n = 60
    rng = np.random.default_rng(len(sizes))
    g = {"n_nodes": n + 1, "edge_u": np.arange(n), "edge_v": np.arange(1, n + 1), "source": 0,
         "sink": n}
    lower, upper = _rows(rng, 900, 900, n, 2, 12)
    refs = R.Refs(rsr_ctx, n, 2, lower, upper)
    system = R.System(rsr_ctx, g)
    model = R.Model(rsr_ctx, _model(n, 2, 12))
    jobs = [{"model": model, "refs": refs, "system": system, "seed": 50 + k, "N": N, "grad": False,
             "buffers": R.Buffers(rsr_ctx, n, 2, N)} for k, N in enumerate(sizes)]
    plan = R.Plan(rsr_ctx, jobs, tune=False)
    plan.run()
    plan.results(want_grad=False)
    for k, job in enumerate(jobs):
        b = job["buffers"]
        want = R.rsr_classify(rsr_ctx, refs, b.samples, job["N"], form=R.RSR_POPCOUNT)
        assert torch.equal(b.flags, want), k
    plan.close()


def test_small_jobs_do_not_slow_a_large_one(rsr_ctx):
    """One large job among 200 small ones against as many samples in one job: about
    twice the time (the jobs' counts), not the many times that a range of tiles
    padded to the largest job takes, whose few full ones fall to a few blocks."""
    n = 240
    rng = np.random.default_rng(8)
    g = {"n_nodes": n + 1, "edge_u": np.arange(n), "edge_v": np.arange(1, n + 1), "source": 0,
         "sink": n}
    lower, upper = _rows(rng, 2000, 2000, n, 2, 12)
    refs = R.Refs(rsr_ctx, n, 2, lower, upper)
    system = R.System(rsr_ctx, g)
    model = R.Model(rsr_ctx, _model(n, 2, 12))
    ms = []
    for sizes in ([1_100_000], [1_000_000] + [500] * 200):
        jobs = [{"model": model, "refs": refs, "system": system, "seed": 50 + k, "N": N,
                 "grad": False, "buffers": R.Buffers(rsr_ctx, n, 2, N)}
                for k, N in enumerate(sizes)]
        plan = R.Plan(rsr_ctx, jobs, tune=False)
        best = float("inf")
        for _ in range(5):
            t = time.perf_counter()
            plan.run()
            plan.results(want_grad=False)
            best = min(best, time.perf_counter() - t)
        ms.append(best * 1e3)
        plan.close()
    assert ms[1] < 5 * ms[0], ms


# Match counts: more matches per lane than a flush holds (255), rows past whole
# slices, empty sides, more tiles than CUs, ragged ends.
@pytest.mark.parametrize("n,K,R_L,R_U,N,bits,mode", [
    (20, 2, 1, 2048, 1, 2, R.RSR_COUNT),
    (33, 2, 2049, 63, 129, 3, R.RSR_COUNT),
    (64, 2, 0, 2100, 2049, 1, R.RSR_COUNT),
    (64, 2, 9001, 0, 700, 1, R.RSR_COUNT),
    (40, 3, 9001, 20_003, 3001, 1, R.RSR_COUNT),
    (295, 2, 300, 2111, 40_001, 6, R.RSR_COUNT),
    (1250, 2, 100, 2050, 1500, 5, R.RSR_COUNT),
    (4096, 2, 2060, 65, 500, 5, R.RSR_COUNT),
    (20, 2, 65, 63, 129, 3, R.RSR_COUNT),
    (33, 2, 2065, 63, 5000, 3, R.RSR_LABEL),
    (70, 4, 300, 5000, 4097, 2, R.RSR_LABEL),
])
def test_counts_against_the_oracle(rsr_ctx, n, K, R_L, R_U, N, bits, mode):
    """Rows of no system: both sides match the same samples."""
    rng = np.random.default_rng(n + N + bits)
    lower = np.where(rng.random((R_L, n)) < bits / n, rng.integers(0, K, (R_L, n)), K - 1)
    upper = np.where(rng.random((R_U, n)) < bits / n, rng.integers(0, K, (R_U, n)), 0)
    lower[:, 1], upper[:, 0] = K - 2, 1      # no row without a bit
    lower, upper = lower.astype(np.uint8), upper.astype(np.uint8)
    model = R.Model(rsr_ctx, np.full((n, K), 1.0 / K))
    refs = R.Refs(rsr_ctx, n, K, lower, upper)
    if mode == R.RSR_LABEL:
        assert not refs.consistent
    xs = R.rsr_sample(rsr_ctx, model, 31, 0, 0, N)
    want, wl, wu = oracle.classify(lower, upper, unpack_states(xs.cpu().numpy(), n, K),
                                   mode=1 if mode == R.RSR_COUNT else 0)
    got = R.rsr_classify(rsr_ctx, refs, xs, N, mode=mode)
    np.testing.assert_array_equal(got.cpu().numpy(), want)
    if mode == R.RSR_COUNT:
        flags, match = R.rsr_classify(rsr_ctx, refs, xs, N, mode=mode, want_match=True)
        np.testing.assert_array_equal(flags.cpu().numpy(), want)
        np.testing.assert_array_equal(match.cpu().numpy()[:, 0], wl)
        np.testing.assert_array_equal(match.cpu().numpy()[:, 1], wu)
        if R_U > 20_000:
            assert int(match[:, 1].max()) > 255 * 16 * 4


# The same on the rows that the automatic form counts this way at any number of
# samples.
@pytest.mark.parametrize("n,K,R_L,R_U,N,bits,mode", [
    (20, 2, 1, 8192, 1, 2, R.RSR_COUNT),
    (33, 2, 8193, 63, 129, 3, R.RSR_COUNT),
    (64, 2, 0, 8300, 2049, 1, R.RSR_COUNT),
    (295, 2, 300, 8511, 40_001, 6, R.RSR_COUNT),
    (1250, 2, 100, 2050, 1500, 5, R.RSR_COUNT),
    (120, 2, 2050, 40, 530_000, 3, R.RSR_COUNT),
    (40, 3, 4097, 20, 1000, 2, R.RSR_COUNT),
    (33, 2, 10_257, 63, 5000, 3, R.RSR_LABEL),
    (340, 3, 300, 10_900, 40_003, 3, R.RSR_LABEL),
    (300, 2, 2065, 63, 525_000, 3, R.RSR_LABEL),
])
def test_counts_of_many_rows(rsr_ctx, n, K, R_L, R_U, N, bits, mode):
    rng = np.random.default_rng(n + N + bits)
    lower = np.where(rng.random((R_L, n)) < bits / n, rng.integers(0, K, (R_L, n)), K - 1)
    upper = np.where(rng.random((R_U, n)) < bits / n, rng.integers(0, K, (R_U, n)), 0)
    lower[:, 1], upper[:, 0] = K - 2, 1      # no row without a bit
    lower, upper = lower.astype(np.uint8), upper.astype(np.uint8)
    model = R.Model(rsr_ctx, np.full((n, K), 1.0 / K))
    refs = R.Refs(rsr_ctx, n, K, lower, upper)
    assert mode == R.RSR_COUNT or not refs.consistent
    xs = R.rsr_sample(rsr_ctx, model, 31, 0, 0, N)
    if N > 100_000:  # the oracle on the first samples, the other form on all
        want = R.rsr_classify(rsr_ctx, refs, xs, N, mode=mode, form=R.RSR_MFMA_FP4,
                              want_match=mode == R.RSR_COUNT)
        got = R.rsr_classify(rsr_ctx, refs, xs, N, mode=mode, want_match=mode == R.RSR_COUNT)
        for a, b in zip(*((got, want) if mode == R.RSR_COUNT else ((got,), (want,)))):
            assert torch.equal(a, b)
    some = min(N, 2000)
    x = unpack_states(xs[:, :some].cpu().numpy(), n, K)
    want, wl, wu = oracle.classify(lower, upper, x, mode=1 if mode == R.RSR_COUNT else 0)
    if mode == R.RSR_COUNT:
        flags, match = R.rsr_classify(rsr_ctx, refs, xs, N, mode=mode, want_match=True)
        np.testing.assert_array_equal(match.cpu().numpy()[:some, 0], wl)
        np.testing.assert_array_equal(match.cpu().numpy()[:some, 1], wu)
    else:
        flags = R.rsr_classify(rsr_ctx, refs, xs, N, mode=mode)
    np.testing.assert_array_equal(flags.cpu().numpy()[:some], want)


def _times(ctx, refs, xs, N, mode, forms):
    us = {}
    for form in forms:
        flags = R.rsr_classify(ctx, refs, xs, N, mode=mode, form=form)
        best = float("inf")
        for _ in range(5):
            torch.cuda.synchronize()
            t = time.perf_counter()
            for _ in range(20):
                R.rsr_classify(ctx, refs, xs, N, mode=mode, form=form, flags=flags)
            torch.cuda.synchronize()
            best = min(best, (time.perf_counter() - t) * 5e4)
        us[form] = best
    return us


@pytest.mark.parametrize("n,rows,N,mode", [
    (40, 2048, 70_000, R.RSR_COUNT), (120, 2100, 200_000, R.RSR_COUNT),
    (295, 4000, 70_000, R.RSR_COUNT), (295, 4000, 70_000, R.RSR_LABEL),
    (640, 2048, 70_000, R.RSR_LABEL), (120, 8000, 70_000, R.RSR_LABEL)])
def test_few_rows_take_the_matrix_cores(rsr_ctx, n, rows, N, mode):
    """Rows of few bits, too few of them to pay for bit-sliced counters (1.2 to 4
    times the FP4 form's time): the automatic form takes no longer than FP4."""
    rng = np.random.default_rng(n)
    lower = np.where(rng.random((rows, n)) < 0.01, 0, 1).astype(np.uint8)
    upper = np.where(rng.random((rows, n)) < 0.01, 1, 0).astype(np.uint8)
    lower[:, 1], upper[:, 0] = 0, 1
    refs = R.Refs(rsr_ctx, n, 2, lower, upper)
    assert not refs.consistent
    model = R.Model(rsr_ctx, np.tile([0.05, 0.95], (n, 1)))
    xs = R.rsr_sample(rsr_ctx, model, 31, 0, 0, N)
    us = _times(rsr_ctx, refs, xs, N, mode, (R.RSR_AUTO, R.RSR_MFMA_FP4))
    assert us[R.RSR_AUTO] < 1.2 * us[R.RSR_MFMA_FP4], us


@pytest.mark.parametrize("n,rows", [(20, 5), (20, 16), (120, 6), (1250, 3)])
def test_few_rows_and_many_samples_take_the_cascade(rsr_ctx, n, rows):
    """A handful of rows on 1e6 samples: no slower than one round of plain tests."""
    rng = np.random.default_rng(n)
    lower, upper = _rows(rng, rows, rows, n, 2, 4)
    refs = R.Refs(rsr_ctx, n, 2, lower, upper)
    assert refs.consistent
    N = 1_000_000
    xs = R.rsr_sample(rsr_ctx, R.Model(rsr_ctx, _model(n, 2, 4)), 31, 0, 0, N)
    us = _times(rsr_ctx, refs, xs, N, R.RSR_LABEL, (R.RSR_AUTO, R.RSR_POPCOUNT))
    assert us[R.RSR_AUTO] < 1.18 * us[R.RSR_POPCOUNT], us
