"""A plan's counts where they can go wrong: jobs of several sizes in one
segment (N below one load, odd, below and above a block's share), flags and Y
at odd addresses, jobs with and without a gradient, several segments, and
replays after other work on the buffers.  Counts, probabilities and gradients
are compared with the oracle's pass over each job."""
import numpy as np
import pytest
import torch

import oracle
import paper_2604_17066_amd as R
import workloads as WL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grads", ["all", "none", "some"])
@pytest.mark.parametrize("sizes,shift", [((7, 4097, 20_000), 0), ((15, 16, 17, 70_001), 1),
                                         ((65_536, 4_096), 3)])
def test_counts_and_gradients(rsr_ctx, grads, sizes, shift):
    a = WL.configs.tiny(N=10)
    b = WL.configs.graph2(N=1, R_U=60, R_L=60)
    jobs, want = [], []
    for c, keep in ((a, 9), (b, 60)):
        lower, upper = c["lower"][:-3][:keep], c["upper"][:-4][:keep]
        model = R.Model(rsr_ctx, c["p"])
        refs = R.Refs(rsr_ctx, c["n"], c["K"], lower, upper)
        system = R.System(rsr_ctx, c["graph"])
        for k, N in enumerate(sizes):
            buf = R.Buffers(rsr_ctx, c["n"], c["K"], N)
            buf.flags = torch.empty(N + 16, dtype=torch.uint8, device=rsr_ctx.device)[shift:shift + N]
            buf.Y = torch.empty(N + 16, dtype=torch.uint8, device=rsr_ctx.device)[shift:shift + N]
            grad = grads == "all" or (grads == "some" and k % 2 == 0)
            jobs.append({"model": model, "refs": refs, "system": system, "seed": 5 + k, "N": N,
                         "buffers": buf, "grad": grad})
            x = oracle.sample(c["p"], 5 + k, 0, 0, N)
            flags, _, _ = oracle.classify(lower, upper, x, mode=0)
            Y, _ = oracle.eval_unknown(c["graph"], x, flags)
            want.append((oracle.counts(flags, Y), oracle.grad(c["p"], x, Y)[1], N))
    plan = R.Plan(rsr_ctx, jobs, tune=False)
    for replay in range(3):
        for j in jobs:
            j["buffers"].flags.fill_(1)
            j["buffers"].Y.fill_(1)
            j["buffers"].G.fill_(-1.0)
        plan.run()
        ests, gs = plan.results()
        for k, (cnt, G, N) in enumerate(want):
            got = [ests[k][key] for key in ("n_L", "n_U", "n_u", "n_both", "n_u_up")]
            assert got == [int(v) for v in cnt[:5]], (replay, k)
            assert ests[k]["P"] == (got[1] + got[4]) / N
            if jobs[k]["grad"]:
                np.testing.assert_allclose(gs[k], G, rtol=1e-5, atol=0)
                np.testing.assert_array_equal(jobs[k]["buffers"].G.cpu().numpy(), gs[k])
