"""The line searches of a wave's groups, which share the wave's lanes once half
of the groups have their step: requests of different dimensions, trial counts
and start counts in one launch, so that the groups of a wave search together
with different limits, and a tolerance no start reaches, so that starts stall
(every trial of every search fails) and few of them are left at the end.
Against the oracle, bit for bit: the sums a trial forms do not depend on the
lanes that form them."""
import numpy as np
import pytest

from paper_2603_28770_amd import workloads as W

pytestmark = pytest.mark.gpu

KEYS = ("f", "x", "iters", "status", "ls_trials", "skips", "resets")


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


# (objective, dimensions that share a group size, L-BFGS pairs)
CASES = [("rastrigin", (3, 4), 0), ("ackley", (1, 2, 3, 4), 0), ("rastrigin", (5, 8), 0),
         ("ackley", (9, 16), 0), ("rastrigin", (17, 32), 0), ("rosenbrock", (33, 64), 0), ("rosenbrock", (2, 4), 0),
         ("rastrigin", (1, 3, 4), 5), ("ackley", (5, 8), 8), ("rosenbrock", (9, 16), 1),
         ("rastrigin", (17, 32), 3), ("rosenbrock", (33, 64), 8), ("ackley", (65, 128), 4),
         ("rastrigin", (129, 256), 8)]


@pytest.mark.parametrize("objective,dims,m", CASES, ids=lambda v: str(v).replace(" ", ""))
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_shared_searches(Z, ctx, oracle_mod, objective, dims, m, precision):
    lo, hi = W.BOXES[objective]
    # few trials let the polynomial objective run off to infinity
    few, some = (12, 25) if objective == "rosenbrock" else (1, 5)
    ps = [W.problem(objective=objective, dim=d, n=n, lower=lo, upper=hi, iter_pso=2, iter_bfgs=40,
                    iter_ls=ls, grad_tol=1e-150, seed=7, request_id=10 * i + k, lbfgs_m=m,
                    precision=precision)
          for i, d in enumerate(dims) for k, (n, ls) in enumerate(((1, 20), (6, few), (3, some), (5, 40)))]
    print(f"\n[search] {objective} {dims} m={m} {precision}", flush=True)
    got = Z.zeus_minimize_batch(ctx, ps)
    for p, g in zip(ps, got):
        alone = Z.zeus_minimize(ctx, p)  # the same start in a wave of its own
        for k in KEYS:
            assert np.array_equal(g[k], alone[k], equal_nan=g[k].dtype.kind == "f"), (p, k)
        if precision == "fp64":
            o = oracle_mod.bfgs(p, oracle_mod.pso(p)["x"])
            for k in KEYS:
                assert np.array_equal(g[k], o[k], equal_nan=g[k].dtype.kind == "f"), (p, k)
