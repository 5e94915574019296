"""The gradient's counts where they can go wrong: one block and the most blocks
a word takes, one component and several words, several planes, the most padded
bits (257 components of 16 states: 4320 bits for 3855), Y all zero and all one,
repeated calls, and the importance from the same partials.  Counts and results
are compared with the oracle's."""
import numpy as np
import pytest
import torch

import oracle
import paper_2604_17066_amd as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,K,N", [(1, 2, 1), (1, 16, 300), (32, 2, 16_384), (33, 3, 16_385),
                                   (295, 2, 50_001), (64, 4, 200_003), (5, 2, 1_032_193),
                                   (257, 16, 1_032_193)])
def test_counts_and_results(rsr_ctx, n, K, N):
    rng = np.random.default_rng([n, K, N])
    p = rng.dirichlet(np.full(K, 1.5), size=n)
    p[0, 0] = 0.0
    p[0] /= p[0].sum()
    model = R.Model(rsr_ctx, p)
    xs = R.rsr_sample(rsr_ctx, model, 21, 0, 0, N)
    x = oracle.sample(p, 21, 0, 0, N)
    for k, y in enumerate((rng.integers(0, 2, N), np.zeros(N), np.ones(N), rng.integers(0, 2, N))):
        Y = y.astype(np.uint8)
        G, counts = R.rsr_grad(rsr_ctx, model, xs, torch.from_numpy(Y).to(rsr_ctx.device), N,
                               want_counts=True)
        torch.cuda.synchronize()
        want_c, want_G = oracle.grad(p, x, Y)
        np.testing.assert_array_equal(counts.cpu().numpy().view(np.uint64), want_c, err_msg=str(k))
        np.testing.assert_allclose(G.cpu().numpy().astype(np.float64), want_G, rtol=1e-5, atol=0)
        if K == 2:
            I = R.rsr_importance(rsr_ctx, model, xs, torch.from_numpy(Y).to(rsr_ctx.device), N)
            torch.cuda.synchronize()
            with np.errstate(divide="ignore", invalid="ignore"):
                q = np.where(p > 0, want_c / (N * p), 0.0)
            np.testing.assert_array_equal(I.cpu().numpy(), (q[:, 1] - q[:, 0]).astype(np.float32))
        if N > 1_000_000 and k == 1:
            break
