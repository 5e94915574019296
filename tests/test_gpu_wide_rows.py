"""LABEL classification of more than 2048 packed bits with dense rows (the
popcount cascade; the other forms take sparse rows or fewer bits): 65 to 96
words share one instantiation, whose tile of rows is the only one that 4096
words do not fill in whole groups of 8."""
import numpy as np
import pytest

import oracle
import paper_2604_17066_amd as R
from helpers import unpack_states

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,K,R_L,R_U", [
    (2050, 2, 41, 48),       # one tile and its last rows
    (2500, 2, 300, 700),
    (3072, 2, 83, 2),
    (136, 16, 90, 0),
    (3073, 2, 200, 300),     # the next instantiation
])
def test_dense_rows_of_many_words(rsr_ctx, n, K, R_L, R_U):
    rng = np.random.default_rng(n + R_L)
    N = 2500
    model = R.Model(rsr_ctx, np.full((n, K), 1.0 / K))
    xs = R.rsr_sample(rsr_ctx, model, 21, 0, 0, N)
    x = unpack_states(xs.cpu().numpy(), n, K)
    # Rows just above and just below drawn samples.  Component 0 keeps them
    # consistent.
    low_of = np.flatnonzero(x[:, 0] < K - 1)[:R_L]
    up_of = np.flatnonzero(x[:, 0] == K - 1)[:R_U]
    lower, upper = x[low_of].copy(), x[up_of].copy()
    lower[rng.random(lower.shape) < 0.1] = K - 1
    upper[rng.random(upper.shape) < 0.1] = 0
    lower[:, 0], upper[:, 0] = K - 2, K - 1
    refs = R.Refs(rsr_ctx, n, K, lower, upper)
    assert refs.consistent
    want, _, _ = oracle.classify(lower, upper, x, mode=0)
    assert (want[low_of] == 1).all() and (want[up_of] == 2).all() and (want == 0).any()
    for form in (R.RSR_AUTO, R.RSR_POPCOUNT):
        got = R.rsr_classify(rsr_ctx, refs, xs, N, form=form)
        np.testing.assert_array_equal(got.cpu().numpy(), want, err_msg=f"form {form}")
