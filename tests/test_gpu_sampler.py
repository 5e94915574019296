"""The sampler against the oracle where its compares can go wrong: thresholds
whose high half is 0, 1 or 65535, with and without low bits, sure and
impossible states, words that are split over blocks, ragged component counts
and a sample range that crosses a multiple of 2^32."""
import numpy as np
import pytest

import oracle
from helpers import pad_bits, unpack_states

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 65535, 65536, 65537, 131071, 131072, 131073, 2 ** 31, 2 ** 32 - 65537,
         2 ** 32 - 65536, 2 ** 32 - 65535, 2 ** 32 - 1, 2 ** 32]


def _binary(n, thresholds):
    c = np.resize(np.array(thresholds, dtype=np.float64), n)
    return np.stack([c / 2 ** 32, 1.0 - c / 2 ** 32], axis=1)


CASES = {
    "one component": (_binary(1, [2 ** 31 + 1]), 0, 70_000),
    "threshold edges": (_binary(40, EDGES), 0, 400_000),
    "edges in one block": (_binary(8, EDGES[:8]), 5, 300_001),
    "upper edges in one block": (_binary(9, EDGES[5:]), 5, 300_001),
    "forced beside decided words": (_binary(97, [7 * 2 ** 28] * 40 + [3] + [2 ** 31] * 56), 0, 50_003),
    "thresholds below 2^16 in every block": (_binary(33, [1, 2 ** 31, 65535, 40_000, 2 ** 28]), 1,
                                             600_001),
    "rare states of several levels": (np.tile([[2 / 2 ** 32, 60_000 / 2 ** 32, 65_536 / 2 ** 32,
                                                1 - 125_538 / 2 ** 32],
                                               [0.0, 9_000 / 2 ** 32, 0.5, 0.5 - 9_000 / 2 ** 32]],
                                              (20, 1)), 0, 500_000),
    "few samples, many words": (_binary(1250, [2 ** 30 + 12345, 2 ** 29, 2 ** 31 + 7]), 0, 130),
    "across 2^32": (_binary(70, [2 ** 30 + 1, 2 ** 31]), 2 ** 32 - 101, 1000),
    "three states": (np.tile([[3 / 2 ** 32, 0.25, 0.75 - 3 / 2 ** 32], [0.0, 0.5, 0.5],
                              [2 ** -16, 2 ** -15, 1 - 2 ** -16 - 2 ** -15], [1.0, 0.0, 0.0]], (9, 1)),
                     0, 200_000),
    "sixteen states": (np.full((21, 16), 1 / 16), 3, 60_000),
}


@pytest.mark.parametrize("name", list(CASES))
def test_states_equal_the_oracle(rsr_ctx, name):
    import paper_2604_17066_amd as R
    p, first, N = CASES[name]
    model = R.Model(rsr_ctx, p)
    words = R.rsr_sample(rsr_ctx, model, 0x123456789ABCDEF0, 9, first, N).cpu().numpy()
    assert pad_bits(words, *p.shape) == 0
    assert np.array_equal(unpack_states(words, *p.shape),
                          oracle.sample(p, 0x123456789ABCDEF0, 9, first, N))


def _time_us(fn, reps=20):
    import torch
    best = float("inf")
    for _ in range(5):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(reps):
            fn()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / reps)
    return best


@pytest.mark.parametrize("K", [2, 3])
def test_rare_states_cost_no_more(rsr_ctx, K):
    """Components that fail with probability 1e-6 (or some of them) are drawn about
    as fast as ones that fail with 0.01: few samples need the second block."""
    import paper_2604_17066_amd as R
    n, N = 295, 500_000
    times = []
    for fail in (np.full(n, 0.01), np.full(n, 1e-6), np.full(n, 2.0 ** -16),
                 np.where(np.arange(n) % 32 == 7, 5e-6, 0.05)):
        p = np.repeat(fail[:, None] / (K - 1), K, axis=1)
        p[:, K - 1] = 1.0 - fail
        model = R.Model(rsr_ctx, p)
        out = R.rsr_sample(rsr_ctx, model, 5, 0, 0, N)
        times.append(_time_us(lambda: R.rsr_sample(rsr_ctx, model, 5, 0, 0, N, out=out)))
    # Redrawing every block of every sample takes about three times as long.
    assert max(times[1:]) < 1.6 * times[0], times
