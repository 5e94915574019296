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
