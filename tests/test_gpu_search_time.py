"""Times of line searches that must not depend on what a search does not do.
Ratios of two times of the same device and process, each the best of several
solves taken in turn, with limits between what the two sides measure when they
do the same work and when they do not."""
import time

import pytest

from paper_2603_28770_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def Z():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_28770_amd import zeus
    return zeus


@pytest.fixture(scope="module")
def ctx(Z):
    c = Z.zeus_context_create(0)
    yield c
    Z.zeus_context_destroy(c)


def _best(Z, ctx, problems, reps=7):
    """The shortest time of each problem (device entry), the problems in turn."""
    import torch
    runs = [Z.DeviceSolve(p) for p in problems]
    best = [float("inf")] * len(runs)
    for rep in range(reps + 1):
        for k, r in enumerate(runs):
            torch.cuda.synchronize()
            t = time.perf_counter()
            r.enqueue(ctx)
            torch.cuda.synchronize()
            if rep:
                best[k] = min(best[k], time.perf_counter() - t)
    return best


@pytest.mark.parametrize("d", [3, 4])
def test_no_step_lengths_past_the_last_trial(Z, ctx, d):
    # a start that takes its sixth or seventh trial at every step has the 64
    # lanes of its wave for the second round: with 20 trials a search the step
    # lengths come from the table of 32, with 68 they go on to the 68th
    p = W.problem(objective="rastrigin", dim=d, n=1, lower=-5.12, upper=5.12, iter_pso=1,
                  iter_bfgs=3000, grad_tol=1e-150, seed=4)
    t20, t68 = _best(Z, ctx, [dict(p, iter_ls=20), dict(p, iter_ls=68)])
    print(f"\n[search time] d={d}: {1e3 * t20:.3f} / {1e3 * t68:.3f} ms", flush=True)
    assert t20 < 0.9 * t68
